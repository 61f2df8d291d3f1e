// Internal layout of a plan: host task list plus the launch tables derived
// from it, and their lazily created device copies.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <limits>
#include <mutex>
#include <vector>

#include "cleave.h"

namespace cleave {

// Workgroup tile classes of the execute kernel.  Which class a task uses is a
// pure function of its record (see tile_class_of), so a re-issued task is cut
// into the same sub-tiles no matter which other tasks share the launch.
enum TileClass : int { kTileLarge = 0, kTileSmall = 1, kNumTileClasses = 2 };

#ifndef CLEAVE_LARGE_TILE_ROWS
#define CLEAVE_LARGE_TILE_ROWS 256
#endif
#ifndef CLEAVE_LARGE_TILE_COLS
#define CLEAVE_LARGE_TILE_COLS 256
#endif
constexpr int kLargeTileRows = CLEAVE_LARGE_TILE_ROWS;
constexpr int kLargeTileCols = CLEAVE_LARGE_TILE_COLS;
constexpr int kSmallTileRows = 128;
constexpr int kSmallTileCols = 128;

__host__ __device__ inline int tile_rows(int cls) { return cls == kTileLarge ? kLargeTileRows : kSmallTileRows; }
__host__ __device__ inline int tile_cols(int cls) { return cls == kTileLarge ? kLargeTileCols : kSmallTileCols; }

// Blocks with both edges above 128 are cut into large sub-tiles, everything
// else into 128 x 128 ones.
__host__ __device__ inline int tile_class_of(const cleave_task& t) {
  return (t.m_len > 128 && t.n_len > 128) ? kTileLarge : kTileSmall;
}

// One unit of work of the execute kernels: a sub-tile of one task's output
// block, computed over the task's whole chunk of the inner dimension.  The
// record carries everything a workgroup needs, so that one load -- issued well
// ahead -- replaces the dependent pair "which task, then that task's record".
// Elements of K the direct (global -> LDS) execute kernel consumes per step.
constexpr uint32_t kDirectKStep = 64;

// Steps of `per_step` elements in a chunk, the last one whole or not.  A chunk has
// up to 2^31 - 1 elements: rounded up in 32 bits without a sign, or the longest
// ones come out negative.
__host__ __device__ constexpr int chunk_steps(uint32_t k_len, uint32_t per_step) {
  return static_cast<int>((k_len + per_step - 1) / per_step);
}

// What the general kernel's launch over a list of tasks is chosen by.
struct ListShape {
  uint32_t longest = 0, shortest = std::numeric_limits<uint32_t>::max();   // chunks
  uint32_t rows = 0, cols = 0;   // most of a block
  int64_t parts64 = 0;           // 64 x 64 parts that the blocks fill or reach into
  void add(const cleave_task& t) {
    longest = t.k_len > longest ? t.k_len : longest;
    shortest = t.k_len < shortest ? t.k_len : shortest;
    rows = t.m_len > rows ? t.m_len : rows;
    cols = t.n_len > cols ? t.n_len : cols;
    parts64 += int64_t{t.m_len / 64 + (t.m_len % 64 != 0)} * (t.n_len / 64 + (t.n_len % 64 != 0));
  }
  // a sixteenth shorter at most: the last chunk of a split that does not divide
  bool equal() const { return uint64_t{16} * shortest >= uint64_t{15} * longest; }
};

struct alignas(16) WorkItem {
  uint32_t m_base, n_base;    // first row / column of the sub-tile in the logical output
  uint32_t k0, k_len;         // the task's chunk
  uint32_t m_valid, n_valid;  // extent of the sub-tile (at most the class's tile)
  uint32_t out_ld;            // row stride of the task's partial block (= its n_len)
  uint32_t gemm_id;           // batch member (batched plans)
  uint64_t out_off;           // element offset of the sub-tile's origin in the partial buffer
  uint32_t task;              // index into the task table
  uint32_t sub;               // sub-tile index within the task's block, row-major
};
static_assert(sizeof(WorkItem) == 48, "WorkItem is 48 bytes");

// How a task's block is cut into sub-tiles: the class (or, with `fine`, the
// small class for every block) fixes the sub-tile, the block's extent the grid
// of sub-tiles.  Host and device share this one definition.
struct SubTiling {
  int cls;
  uint32_t tr, tc;    // sub-tile rows / columns
  uint32_t sm, sn;    // grid of sub-tiles
  __host__ __device__ uint32_t count() const { return sm * sn; }
};
__host__ __device__ inline SubTiling sub_tiling(const cleave_task& t, bool fine) {
  SubTiling s;
  s.cls = fine ? static_cast<int>(kTileSmall) : tile_class_of(t);
  s.tr = static_cast<uint32_t>(tile_rows(s.cls));
  s.tc = static_cast<uint32_t>(tile_cols(s.cls));
  s.sm = (t.m_len + s.tr - 1) / s.tr;
  s.sn = (t.n_len + s.tc - 1) / s.tc;
  return s;
}
// Work item of sub-tile `sub` (row-major in the grid) of task record t.
__host__ __device__ inline WorkItem make_work_item(const cleave_task& t, uint32_t task_index,
                                                   const SubTiling& s, uint32_t sub) {
  const uint32_t i = sub / s.sn, j = sub - i * s.sn;
  WorkItem w{};
  w.m_base = t.m0 + i * s.tr;
  w.n_base = t.n0 + j * s.tc;
  w.k0 = t.k0;
  w.k_len = t.k_len;
  w.m_valid = s.tr < t.m_len - i * s.tr ? s.tr : t.m_len - i * s.tr;
  w.n_valid = s.tc < t.n_len - j * s.tc ? s.tc : t.n_len - j * s.tc;
  w.out_ld = t.n_len;
  w.gemm_id = t.gemm_id;
  w.out_off = t.partial_off + static_cast<uint64_t>(i) * s.tr * t.n_len + static_cast<uint64_t>(j) * s.tc;
  w.task = task_index;
  w.sub = sub;
  return w;
}

// One unit of work of the reduce kernel: a run of elements of one output tile,
// in the tile's row-major order.  The record carries everything the kernel needs
// from the tile's chunk-0 task.
struct alignas(16) ReduceItem {
  uint64_t partial_off;   // the run's first element in the tile's first block
  uint64_t block;         // elements between two splits' blocks
  uint32_t m0, n0;        // row and column of C where the tile row the run starts in begins
  uint32_t col0;          // the run's first column in that tile row
  uint32_t n_len;         // elements per tile row
  uint32_t count;         // elements of the run
  uint32_t ksplit_cnt;
  uint32_t gemm_id;       // batch member (batched plans)
  uint32_t pad;
};
static_assert(sizeof(ReduceItem) == 48, "ReduceItem is 48 bytes");
// The run that starts at element e of the tile whose chunk-0 task is t.
__host__ __device__ inline ReduceItem make_reduce_item(const cleave_task& t, uint64_t e, uint32_t run) {
  ReduceItem item{};
  item.partial_off = t.partial_off + e;
  item.block = static_cast<uint64_t>(t.m_len) * t.n_len;
  item.m0 = t.m0 + static_cast<uint32_t>(e / t.n_len);
  item.n0 = t.n0;
  item.col0 = static_cast<uint32_t>(e % t.n_len);
  item.n_len = t.n_len;
  const uint64_t left = item.block - e;
  item.count = left < run ? static_cast<uint32_t>(left) : run;
  item.ksplit_cnt = t.ksplit_cnt;
  item.gemm_id = t.gemm_id;
  return item;
}
// An output tile as the host lists it: the runs' records, one per run, are
// written when the plan is uploaded, on the device unless the table is short.
// Making them with the plan took longer; creation + upload in us, one 16-byte
// record per 4096 elements / 48-byte records of all runs made with the plan /
// this list, 2048 x 3072 x 768 in 256 x 256 tiles, S = 2 107 / 164 / 154,
// 4096 x 11008 x 4096 in 512 x 512, S = 4 440 / 661 / 450.
struct ReduceTile {
  uint32_t task;    // the tile's chunk-0 task
  uint32_t run;     // elements per run
  uint64_t first;   // the first run's place in the table
};

// Tables of the returned-block check.  A row segment is a distinct (m0, m_len)
// of the task list, a column segment a distinct (n0, n_len): the projections
// of A onto r and of B onto s are computed once per segment and shared by all
// tasks that use it.
struct Segment {
  uint32_t start, len;
};
// One unit of work of the bilinear-form kernels: a run of rows of one task's
// partial block, or (fused pass) of all splits' blocks of a tile.  The record
// carries everything the kernels need from the (first split's) task.
struct alignas(16) VerifyItem {
  uint64_t partial_off;     // first element of the run in the (first split's) block
  uint64_t block;           // fused pass: elements between two splits' blocks
  uint32_t m0, n0;          // first row and column of the run in the output
  uint32_t n_len;           // elements per row
  uint32_t count;           // elements of the run
  uint32_t gemm_id;         // batch member
  uint32_t ksplit_cnt;      // fused pass: splits of the tile,
  uint32_t slot, slot_step; // where the sum of its first split goes, and how much further on the next one's
};
static_assert(sizeof(VerifyItem) == 48, "VerifyItem is 48 bytes");
inline VerifyItem make_verify_item(const cleave_task& t, uint32_t row0, uint32_t rows) {
  VerifyItem item{};
  item.partial_off = t.partial_off + static_cast<uint64_t>(row0) * t.n_len;
  item.block = static_cast<uint64_t>(t.m_len) * t.n_len;
  item.m0 = t.m0 + row0;
  item.n0 = t.n0;
  item.n_len = t.n_len;
  item.count = rows * t.n_len;
  item.gemm_id = t.gemm_id;
  item.ksplit_cnt = t.ksplit_cnt;
  return item;
}

struct VerifyTables {
  std::vector<Segment> row_segs, col_segs;
  std::vector<uint32_t> task_row_seg, task_col_seg;   // per task
  std::vector<VerifyItem> items;                      // a task's items are adjacent
  std::vector<uint32_t> task_first_item;              // n_tasks + 1 entries
  // Fused check + aggregation: its own, shorter items (runs of rows of a tile,
  // taken for all splits at once; listed for the first split's task only) and
  // the slots their sums go to (a task's slots are adjacent, as above).
  std::vector<VerifyItem> agg_items;
  std::vector<uint32_t> agg_first_item;               // n_tasks + 1 entries
  uint32_t max_ksplit = 1;
  bool segs_mult8 = true;   // every segment start and length a multiple of 8
  bool segs_mult4 = true;
  // device copies and scratch (allocated once, on the device the plan lives on)
  Segment* d_row_segs = nullptr;
  Segment* d_col_segs = nullptr;
  uint32_t* d_task_row_seg = nullptr;
  uint32_t* d_task_col_seg = nullptr;
  VerifyItem* d_items = nullptr;
  uint32_t* d_task_first_item = nullptr;
  VerifyItem* d_agg_items = nullptr;
  uint32_t* d_agg_first_item = nullptr;
  double* d_agg_item_sums = nullptr;
  double* d_proj = nullptr;       // U, |U| (row segs x K each), V, |V| (col segs x K each)
  double* d_item_sums = nullptr;  // one per item
};

// Device memory the subset launches of a plan put their work-item lists in.
// Sized when the plan's tables are uploaded; nothing is allocated later.
//   eager calls:    slices of a ring of 2 * max_items items; a slice is reused
//                   only after the launch that read it has finished (one event
//                   per launch; the host waits only if the ring has wrapped
//                   onto a launch that is still running);
//   captured calls: (the stream is being captured into a HIP graph) slices of a
//                   second buffer of max_items items that are never reused,
//                   since a graph may be replayed as long as the plan lives.
// max_items = the plan's own work-item count under its finest cut, which no
// subset exceeds.
struct SubsetRing {
  WorkItem* d_ring = nullptr;
  WorkItem* d_captured = nullptr;
  int64_t max_items = 0;
  int64_t pos = 0;             // next free item of the ring
  int64_t captured_used = 0;   // items of d_captured handed out
  struct InFlight {
    int64_t begin, end;
    hipEvent_t done;
  };
  std::vector<InFlight> in_flight;       // oldest first
  std::vector<hipEvent_t> idle_events;
  std::mutex mu;                         // subset calls of one plan may come from several threads
};

// Appends the work items of `task_index` (record t) to out[class].  With
// `fine` every block is cut into small-class sub-tiles.  Either cut gives the
// same bits: both kernels shapes accumulate an output element in the same
// order (ascending K steps and sub-steps), so the choice is free per launch.
// Workgroup schedule for a list of work items of unequal length (heterogeneous
// tilings: Sec. 4.1 gives every device its own shard size, Sec. 3.2 its own
// split of the inner dimension).  The persistent kernel's default -- workgroup
// b takes items b, b + grid, ... -- leaves the workgroups with very different
// totals when chunk lengths differ by a factor of eight.  This reorders the
// items so that workgroup b owns the contiguous run
// [ranges[b], ranges[b + 1]) and the runs have nearly equal cost: longest items
// first, each to the least-loaded workgroup of the XCD the item's position
// belongs to (position mod 8, as the list was laid out) unless a workgroup of
// another XCD is behind by more than a quarter of the item's own cost; inside a
// run the original order is kept.  Largest load over the mean with a whole item
// as the limit / a quarter, a 4096 x 11008 x 4096 tiling: large class 1.38 /
// 1.16, small class 1.78 / 1.37.  Nothing and a half give the same as a quarter,
// and over 150 lists of 25 drawn problems the mean hardly moves (3.39 / 3.36):
// in most of them one item is longer than a workgroup's share.  Returns with
// `ranges` empty, and the list untouched, when no two items differ by more than a
// K step or so (the last chunk of a split that does not divide: every workgroup
// meets as many of those) or no workgroup gets a second item.
bool needs_balance(const std::vector<WorkItem>& items, int grid);
void balance_work_items(std::vector<WorkItem>& items, int grid, std::vector<uint32_t>* ranges);
// The balanced schedule as it is uploaded.  The runs are the persistent kernel's
// alone; the general kernel takes position i of a list on XCD i % 8, where the
// items as they were laid out share operands.  A list that both kernels run
// (`both`) therefore keeps its order, and the balanced one follows it.  us, the
// general kernel on heterogeneous tilings in the order of the runs / as laid out:
// bf16 with unaligned rows, 4096 x 11008 x 4096 1024 / 739, 5064 x 3080 x 6472
// 528 / 440, 1096 x 2312 x 7304 114 / 115; fp32, 4096^3 1306 / 1157, 2056 x 4104 x
// 4104 720 / 631; the other way round where few items are far longer than the
// rest: bf16 1224 x 4872 x 5384 178 / 193, fp32 2048 x 2048 x 8192 619 / 648.
// Empty, with no ranges, where the list needs no balance.
std::vector<WorkItem> scheduled_list(const std::vector<WorkItem>& items, int grid, bool both,
                                     std::vector<uint32_t>* ranges);
// Cost of a work item in the schedule's unit (one K step of the fast kernel):
// its K steps plus a constant for the store phase (measured: 12 K clocks
// against 2.6 K per step).
inline double work_item_cost(const WorkItem& w) {
  return chunk_steps(w.k_len, kDirectKStep) + 4.5;
}

void append_work_items(const cleave_task& t, uint32_t task_index, std::vector<WorkItem>* out,
                       bool fine = false);

}  // namespace cleave

struct cleave_plan {
  int64_t M = 0, N = 0, K = 0;
  int64_t partial_elems = 0;
  int64_t num_tiles = 0;
  int64_t batch = 0;         // > 0: a batch of that many M x N x K GEMMs, task.gemm_id = member
  int64_t uniform_splits = 0;   // plain plans whose tiles all have that many splits (0: others)
  bool all_k_mult8 = true;   // every k0 and k_len is a multiple of 8
  bool all_m_mult8 = true;   // every m0 and m_len is a multiple of 8
  bool all_n_mult8 = true;   // every n0 and n_len is a multiple of 8
  bool chunk_tails = false;  // some k_len is no multiple of the direct kernel's K step
  int64_t min_k_end = std::numeric_limits<int64_t>::max();   // smallest k0 + k_len of a task
  cleave::ListShape shape;   // of all tasks
  bool all_n_mult4 = true;   // every n0, n_len multiple of 4 (vector path of reduce)
  std::vector<cleave_task> tasks;
  // All tasks, launch order.
  std::vector<cleave::WorkItem> items[cleave::kNumTileClasses];
  // All tasks cut into small-class sub-tiles only: used when the large class
  // would leave too many of the CUs without a work item (cut_small in api.cpp).
  std::vector<cleave::WorkItem> items_fine;
  // Whole K steps of the items of the three lists (large, small, fine), together.
  int64_t items_steps[cleave::kNumTileClasses + 1] = {0, 0, 0};
  // K steps of the longest and of the shortest large item, the last one whole or not.
  int large_steps = 0, large_steps_least = std::numeric_limits<int>::max();
  std::vector<cleave::ReduceTile> reduce_tiles;
  int64_t reduce_runs = 0;

  // Device copies (current device at first use).
  int device = -1;
  cleave_task* d_tasks = nullptr;
  cleave::WorkItem* d_items[cleave::kNumTileClasses] = {nullptr, nullptr};
  cleave::WorkItem* d_items_fine = nullptr;
  // Balanced schedules of the three lists (large, small, fine) for
  // the grid sizes of the device the tables were uploaded to; null = equal items,
  // or a list that the persistent kernel does not run.  The items in balanced order
  // replace those of the first two lists, and stand behind those of the third.
  uint32_t* d_wg_ranges[cleave::kNumTileClasses + 1] = {nullptr, nullptr, nullptr};
  int wg_ranges_grid[cleave::kNumTileClasses + 1] = {0, 0, 0};
  cleave::ReduceItem* d_reduce_items = nullptr;   // reduce_runs records (and behind them what they were made from)
  // Work-item slices of subset launches (device memory sized once, at upload).
  cleave::SubsetRing subset;
  // Repeat check of a subset's task ids without clearing or allocating: task i
  // was listed in the current call iff seen_stamp[i] == seen_generation (one
  // entry per task, made with the plan; guarded by subset.mu).
  std::vector<uint32_t> seen_stamp;
  uint32_t seen_generation = 0;

  // Tables and scratch of the returned-block check; created by its first call.
  cleave::VerifyTables* verify = nullptr;

  const char* last_kernel = "none";
};
