// Host-side task generation: row blocks of A x column blocks of B x chunks of
// the inner dimension (paper Sec. 3.2 "Seamless training", Sec. 4.1 "Search
// space of GEMM"; coverage and zero-task constraints of Sec. 4.1).
#include <algorithm>
#include <cmath>
#include <functional>
#include <limits>
#include <new>
#include <queue>
#include <utility>

#include "plan_internal.h"

namespace cleave {

namespace {

struct Tile {
  int64_t m0, m_len, n0, n_len;
  int32_t ksplit;
};

constexpr int64_t kMaxDim = std::numeric_limits<int32_t>::max();

bool valid_split(int64_t K, int64_t S) {
  if (S < 1 || S > K) return false;
  const int64_t kc = (K + S - 1) / S;
  return (S - 1) * kc < K;
}

constexpr int kXcds = 8;
// A batch member with at least this many work items (one per CU of the chip) is
// spread over all XCDs instead of being kept on one.
constexpr size_t kSpreadItems = 256;

// The work items that run on an XCD at the same time (32 CUs, one large item or two small
// ones on each) are taken from a patch of 4 x 8 (long lists of small items of one GEMM 8 x 8) sub-tiles at one chunk of the
// inner dimension: they share that many row panels of A and column panels of B in the XCD's L2.
// Small items in patches of 4 x 8 / 8 x 8, bf16 in 128 x 128 blocks, the time of the second
// over the first's, operands as the launch before left them / in no cache, layouts NN, NT, TN: 8192^2
// with 128 of K 0.914 / 0.930, 0.918 / 0.931, 0.943 / 0.933, with 1024 0.984 / 0.924, 0.990 / 0.937, 0.960
// / 0.920; 16384 x 4096 x 4096 in 4 splits 0.944 / 0.943, 0.951 / 0.945, 0.959 / 0.961; 6144^2 with 2048
// 0.989 / 0.988, 0.976 / 0.984, 0.966 / 0.972.  Fewer items cover their regions in a few patches
// and gain less or lose: 2048 with 1024 of K 1.002 / 0.955, 0.997 / 0.980, 1.003 / 0.972, with 512 up to
// 1.035 / 1.011, 1024 with 2048 1.003 / 1.001, 1.026 / 1.002, 1.034 / 0.997.  The general kernel,
// which runs this list too: 4096 items, fp32, 8192^2 with 128 of K 0.993 / 0.971, 0.996 / 0.978, 1.002 /
// 0.997, bf16 with unaligned rows 16384 x 4096 with 256 0.981 / 0.974, 0.955 / 0.978, 0.964 / 0.968; both
// 0.97 to 1.03 from 2304 items on with 512 of K and more.
// Large items stay with 4 x 8, which is all that an XCD runs at a time: the second round that 8 x 8
// adds wins or loses with how the patches divide the regions, on both sides of any length of the
// list.  8192 x 12288 with 512 of K (1536 items) 0.993 / 1.038, 1.002 / 1.047, 0.983 / 1.026; 16384 x 8192 with
// 1024 (2048) 1.020 / 1.022, 1.022 / 1.004, 1.024 / 1.014; 9216 x 8448 in 2 splits of 1024 (2376) 0.999 /
// 0.978, 0.974 / 0.980, 0.971 / 0.985; 16384 x 12288 with 512 (3072) 1.049 / 1.026, 1.029 / 1.021, 1.040 / 1.030;
// 8192 x 3072 in 8 splits of 512 (3072) 1.004 / 1.063, 1.007 / 1.001, 1.005 / 1.073; 16384 x 5120 in 8 of 1728
// (10240) 0.984 / 0.988, 0.977 / 0.973, 0.986 / 0.991; three products in a launch, 8192 x 3072 in 2 splits
// of 512 (2304) 1.089 / 1.103, 1.023 / 1.034, 1.094 / 1.089, 4096 x 4096 in 4 of 1024 (3072) 1.047 / 1.047, 1.045 /
// 1.050, 1.102 / 1.051.
constexpr uint32_t kPatchCols = 8;
constexpr size_t kManySmallItems = 2048;
// So do those of several members: where they take turns patch by patch, a larger patch is longer on its way
// to the member that reads the same panels next.  Three products of one A in a launch, 2048 x 2048 in 4 splits
// of 128 0.979 / 1.074, 0.983 / 1.048, 0.980 / 1.085, 1024 x 4096 in 4 of 256 0.986 / 1.142, 0.997 / 1.141,
// 0.993 / 1.125, 4096 x 4096 with 512 of K 1.005 / 0.992, 0.997 / 0.991, 1.019 / 0.974, bf16 with unaligned
// rows 2048 x 2048 in 3 of 171 0.985 / 1.024, 0.987 / 1.040, 0.978 / 1.035; 32 members of 2048 x 2048 x 128
// 1.109 / 1.051, 1.074 / 1.038, 1.081 / 1.035, 64 of 1024 x 1024 x 128 0.997 / 1.003, 0.991 / 0.999, 1.003 / 0.992.
constexpr uint32_t patch_rows(int cls, size_t items, bool members) {
  return cls == kTileLarge || members || items <= kManySmallItems ? 4 : 8;
}

void order_work_items(cleave_plan* p) {
  // Region grid: minimise M/gm + N/gn over gm * gn = 8.
  int gm = 1, gn = kXcds;
  double best = 0.0;
  for (int g = 1; g <= kXcds; g *= 2) {
    const double cost = static_cast<double>(p->M) / g + static_cast<double>(p->N) / (kXcds / g);
    if (g == 1 || cost < best) {
      best = cost;
      gm = g;
      gn = kXcds / g;
    }
  }
  // three lists: the two classes of the mixed cut, then the all-small cut
  std::vector<WorkItem> all[kNumTileClasses], fine[kNumTileClasses];
  size_t n_all[kNumTileClasses] = {}, n_fine = 0;
  for (const cleave_task& t : p->tasks) {
    const SubTiling mixed = sub_tiling(t, false);
    n_all[mixed.cls] += mixed.count();
    n_fine += sub_tiling(t, true).count();
  }
  for (int cls = 0; cls < kNumTileClasses; ++cls) all[cls].reserve(n_all[cls]);
  fine[kTileSmall].reserve(n_fine);
  for (uint32_t i = 0; i < p->tasks.size(); ++i) {
    append_work_items(p->tasks[i], i, all);
    append_work_items(p->tasks[i], i, fine, true);
  }
  for (int list = 0; list < kNumTileClasses + 1; ++list) {
    const int cls = list < kNumTileClasses ? list : kTileSmall;
    const std::vector<WorkItem>& source = list < kNumTileClasses ? all[cls] : fine[kTileSmall];
    std::vector<WorkItem>& ordered = list < kNumTileClasses ? p->items[cls] : p->items_fine;
    ordered.reserve(source.size());
    for (const WorkItem& w : source) {
      p->items_steps[list] += w.k_len / kDirectKStep;
      if (list != kTileLarge) continue;
      p->large_steps = std::max(p->large_steps, chunk_steps(w.k_len, kDirectKStep));
      p->large_steps_least = std::min(p->large_steps_least, chunk_steps(w.k_len, kDirectKStep));
    }
    if (source.empty()) continue;
    const uint32_t tr = static_cast<uint32_t>(tile_rows(cls));
    const uint32_t tc = static_cast<uint32_t>(tile_cols(cls));
    struct Key {
      uint32_t outer_member, split, pm, pn, inner_member, m, n;
      WorkItem item;
    };
    const uint32_t rows = patch_rows(cls, source.size(), p->batch > 0);
    std::vector<Key> lists[kXcds];
    for (auto& l : lists) l.reserve(source.size() / kXcds + 1);
    // Batch members share no output.  Small members (fewer items than the
    // chip has CUs) stay on one XCD each, member g on XCD g mod 8, one after
    // the other.  Large members (the GEMMs of one DAG level) are spread over
    // the XCDs like a single GEMM, and the members take turns patch by patch,
    // so that an operand panel they share is still in L2 for the next one.
    const bool member_per_xcd = p->batch > 0 && source.size() / static_cast<size_t>(p->batch) < kSpreadItems;
    for (const WorkItem& w : source) {
      const cleave_task& t = p->tasks[w.task];
      const uint32_t m = w.m_base;
      const uint32_t n = w.n_base;
      const int rm = static_cast<int>(static_cast<uint64_t>(m) * gm / static_cast<uint64_t>(p->M));
      const int rn = static_cast<int>(static_cast<uint64_t>(n) * gn / static_cast<uint64_t>(p->N));
      // relative position of the chunk inside [0, K): tiles with different
      // split counts still line up by where in K they work
      const uint32_t split = static_cast<uint32_t>(static_cast<uint64_t>(t.k0) * 64 / static_cast<uint64_t>(p->K));
      const int region = member_per_xcd ? static_cast<int>(t.gemm_id % kXcds) : rm * gn + rn;
      lists[region].push_back(Key{member_per_xcd ? t.gemm_id : 0u, split, m / (rows * tr),
                                  n / (kPatchCols * tc), member_per_xcd ? 0u : t.gemm_id, m, n, w});
    }
    size_t longest = 0;
    for (auto& l : lists) {
      std::stable_sort(l.begin(), l.end(), [](const Key& a, const Key& b) {
        if (a.outer_member != b.outer_member) return a.outer_member < b.outer_member;
        if (a.split != b.split) return a.split < b.split;
        if (a.pm != b.pm) return a.pm < b.pm;
        if (a.pn != b.pn) return a.pn < b.pn;
        if (a.inner_member != b.inner_member) return a.inner_member < b.inner_member;
        if (a.m != b.m) return a.m < b.m;
        return a.n < b.n;
      });
      longest = std::max(longest, l.size());
    }
    // Interleave; when a region runs out, the slot is filled from the region
    // that has most left, so the list has no holes.
    size_t pos[kXcds] = {};
    for (size_t i = 0; i < longest; ++i) {
      for (int x = 0; x < kXcds; ++x) {
        int src = x;
        if (pos[src] >= lists[src].size()) {
          size_t most = 0;
          src = -1;
          for (int y = 0; y < kXcds; ++y) {
            const size_t left = lists[y].size() - pos[y];
            if (left > most) {
              most = left;
              src = y;
            }
          }
          if (src < 0) break;
        }
        ordered.push_back(lists[src][pos[src]++].item);
      }
    }
    for (int x = 0; x < kXcds; ++x)
      for (; pos[x] < lists[x].size(); ++pos[x]) ordered.push_back(lists[x][pos[x]].item);
  }
}

// Elements per reduce item of a tile with S splits (a multiple of 1024: 256
// threads, four elements each).  Short runs, one or two loads of every split per
// thread and no loop, start and end a small launch sooner and keep more
// workgroups in flight in a large one; they stop paying where a thread's few
// loads no longer cover a workgroup's start.  us, runs of 4096 / 2048 / 1024
// elements: S = 2, 768 x 3072 6.5 / 4.6 / 5.0, 8192 x 3072 47.1 / 46.3 / 48.0;
// S = 4, 1024 x 1024 4.9 / 3.6 / 3.7, 4096 x 4096 56 / 54 / 52.6, 3001 x 2500
// 28.0 / 26.2 / 24.9; S = 5, 4096 x 4096 80 / - / 74; S = 8, 4096 x 4096
// 107 / 103 / 113, 8192 x 8192 417 / 419 / 443; S = 1 (a copy), 4096 x 4096
// 23.2 / 23.7 / 26.2 and 24.6 in runs of 16384, 1024 x 1024 3.3 against 7.2.
// Splits without a path of their own, runs of 2048 / 1024: S = 3, 1024 x 1024
// 5.0 / 4.8, 768 x 3072 7.6 / 8.4, 8192 x 8192 195 / 187; S = 6, 7.1 / 6.5,
// 13.5 / 15.6, 364 / 346; S = 7, 7.8 / 7.1, 16.1 / 18.0, 417 / 400; S = 9, 9.0 /
// 8.2, 19.9 / 22.0, 522 / 503; S = 16, 24.7 / 17.6, 40.6 / 38.5, 891 / 841: from
// nine splits on the run of eight is kept, although 1024 is the better one at
// most sizes.
uint32_t reduce_run(uint32_t S) {
  if (S == 1) return 4096;
  return S == 2 || S >= 8 ? 2048 : 1024;
}

constexpr int64_t kLongTable = 2048;   // runs

// Emits the task records of `tiles` in canonical order and fills the derived
// tables.  Returns a status code.
// With n_batch > 0 the tile list is emitted n_batch times, once per batch
// member g, with gemm_id = g (tile ids restart, partial offsets run on).
int finish_plan(int64_t M, int64_t N, int64_t K, const std::vector<Tile>& tiles, uint32_t gemm_id,
                cleave_plan** out, int64_t n_batch = 0) {
  cleave_plan* p = new (std::nothrow) cleave_plan;
  if (!p) return CLEAVE_ENOMEM;
  try {
    const uint64_t copies = n_batch > 0 ? static_cast<uint64_t>(n_batch) : 1;
    p->M = M;
    p->N = N;
    p->K = K;
    p->batch = n_batch;
    p->num_tiles = static_cast<int64_t>(tiles.size() * copies);
    uint64_t off = 0;
    uint32_t tile_id = 0;
    // Task, tile and sub-tile indices are 32-bit in the task record and the
    // launch tables, offsets 64-bit: refuse a plan that does not fit rather
    // than wrap.
    constexpr uint64_t kMaxIndex = std::numeric_limits<uint32_t>::max();
    constexpr uint64_t kMaxElems = static_cast<uint64_t>(std::numeric_limits<int64_t>::max()) / 8;
    uint64_t n_tasks = 0;
    for (const Tile& tl : tiles) {
      n_tasks += static_cast<uint64_t>(tl.ksplit);
      const uint64_t subs = static_cast<uint64_t>((tl.m_len + kSmallTileRows - 1) / kSmallTileRows) *
                            static_cast<uint64_t>((tl.n_len + kSmallTileCols - 1) / kSmallTileCols);
      const uint64_t elems = static_cast<uint64_t>(tl.m_len) * static_cast<uint64_t>(tl.n_len);
      if (subs > kMaxIndex || n_tasks > kMaxIndex || elems > kMaxElems / static_cast<uint64_t>(tl.ksplit) ||
          (off += elems * static_cast<uint64_t>(tl.ksplit)) > kMaxElems) {
        delete p;
        return CLEAVE_EINVAL;
      }
    }
    if (n_tasks > kMaxIndex / copies || off > kMaxElems / copies) {
      delete p;
      return CLEAVE_EINVAL;
    }
    off = 0;
    for (uint64_t g = 0; g < copies; ++g) {
    if (n_batch > 0) gemm_id = static_cast<uint32_t>(g);
    tile_id = 0;
    for (const Tile& tl : tiles) {
      const int64_t S = tl.ksplit;
      const int64_t kc = (K + S - 1) / S;
      for (int64_t s = 0; s < S; ++s) {
        cleave_task t{};
        t.gemm_id = gemm_id;
        t.tile_id = tile_id;
        t.m0 = static_cast<uint32_t>(tl.m0);
        t.m_len = static_cast<uint32_t>(tl.m_len);
        t.n0 = static_cast<uint32_t>(tl.n0);
        t.n_len = static_cast<uint32_t>(tl.n_len);
        t.k0 = static_cast<uint32_t>(s * kc);
        t.k_len = static_cast<uint32_t>(std::min(kc, K - s * kc));
        t.ksplit_idx = static_cast<uint32_t>(s);
        t.ksplit_cnt = static_cast<uint32_t>(S);
        t.partial_off = off;
        off += static_cast<uint64_t>(tl.m_len) * static_cast<uint64_t>(tl.n_len);
        p->tasks.push_back(t);
      }
      ++tile_id;
    }
    }
    p->partial_elems = static_cast<int64_t>(off);
    p->seen_stamp.assign(p->tasks.size(), 0u);

    for (const cleave_task& t : p->tasks) {
      const uint32_t k_or = t.k0 | t.k_len;
      p->all_k_mult8 &= (k_or % 8 == 0);
      p->chunk_tails |= (t.k_len % kDirectKStep != 0);
      p->all_m_mult8 &= ((t.m0 | t.m_len) % 8 == 0);
      p->all_n_mult8 &= ((t.n0 | t.n_len) % 8 == 0);
      p->min_k_end = std::min(p->min_k_end, static_cast<int64_t>(t.k0) + t.k_len);
      p->shape.add(t);
      p->all_n_mult4 &= ((t.n0 | t.n_len) % 4 == 0);
    }

    // Launch tables.  Execution order is free (only the task list's order is
    // part of the interface).  Workgroups are dispatched round-robin over the
    // 8 XCDs (workgroup b runs on XCD b % 8, each with its own L2), so work
    // item 8*i + x is the i-th item of XCD x.  Every XCD gets a compact
    // rectangle of the output (a gm x gn grid of regions with gm*gn = 8, chosen
    // to minimise the operand panels a region needs), and walks it chunk index
    // outermost: the items in flight on an XCD then share few row panels of A
    // and column panels of B, at the same chunk of the inner dimension.
    order_work_items(p);

    p->reduce_tiles.reserve(static_cast<size_t>(p->num_tiles));
    for (uint32_t i = 0; i < p->tasks.size(); ++i) {
      const cleave_task& t = p->tasks[i];
      if (t.ksplit_idx != 0) continue;
      const uint32_t run = reduce_run(t.ksplit_cnt);
      p->reduce_tiles.push_back(ReduceTile{i, run, static_cast<uint64_t>(p->reduce_runs)});
      p->reduce_runs += static_cast<int64_t>((static_cast<uint64_t>(t.m_len) * t.n_len + run - 1) / run);
    }
    // A long table lists the last tiles first: what wrote or read the blocks before
    // (the executor, the returned-block check) went through them from the start, so
    // the end is what the Infinity Cache still holds, and going towards the start
    // keeps ahead of what it evicts.  Aggregation behind execute, and both, us, tiles in
    // order / the other way round: 8192 x 3072, S = 2 54.9 / 53.6 and 102.2 / 101.4; 5120^2,
    // S = 4 79.2 / 77.6 and 173.7 / 172.6; 4096 x 11008, S = 4 135.6 / 132.9 and 267.5 /
    // 262.5; 8192^2, S = 4 211.5 / 205.6 and 469 / 462.  With less than some 200 MB of
    // blocks, on both sides of the line, no difference: 2048 x 1024, S = 2 (1024 runs)
    // both 21.1 / 21.1, 2048^2, S = 4 (4096) 30.7 / 30.8, 4096^2, S = 2 (8192) 63.9 / 63.9.
    if (p->reduce_runs >= kLongTable) {
      std::reverse(p->reduce_tiles.begin(), p->reduce_tiles.end());
      uint64_t first = 0;
      for (ReduceTile& tile : p->reduce_tiles) {
        const cleave_task& t = p->tasks[tile.task];
        tile.first = first;
        first += (static_cast<uint64_t>(t.m_len) * t.n_len + tile.run - 1) / tile.run;
      }
    }
  } catch (const std::bad_alloc&) {
    delete p;
    return CLEAVE_ENOMEM;
  }
  *out = p;
  return CLEAVE_OK;
}

}  // namespace

bool needs_balance(const std::vector<WorkItem>& items, int grid) {
  if (grid < 2 || items.size() <= static_cast<size_t>(grid)) return false;   // one item per workgroup at most
  for (size_t i = 1; i < items.size(); ++i)
    if (std::abs(work_item_cost(items[i]) - work_item_cost(items[0])) > 1.0) return true;   // one step: a shorter last chunk
  return false;
}

void balance_work_items(std::vector<WorkItem>& items, int grid, std::vector<uint32_t>* ranges) {
  ranges->clear();
  const size_t n_items = items.size();
  if (!needs_balance(items, grid)) return;

  std::vector<uint32_t> by_cost(n_items);
  for (size_t i = 0; i < n_items; ++i) by_cost[i] = static_cast<uint32_t>(i);
  std::stable_sort(by_cost.begin(), by_cost.end(),
                   [&](uint32_t a, uint32_t b) { return items[a].k_len > items[b].k_len; });
  // The workgroups of each XCD, least loaded (then lowest) first.  (Looking through
  // all of them for every item: 150 lists of 30 heterogeneous tilings 87 ms, 37 so.)
  typedef std::pair<double, uint32_t> Load;
  std::priority_queue<Load, std::vector<Load>, std::greater<Load>> loads[kXcds];
  for (int b = 0; b < grid; ++b) loads[b % kXcds].push({0.0, static_cast<uint32_t>(b)});
  std::vector<uint32_t> owner(n_items), first(static_cast<size_t>(grid) + 1, 0u);
  for (uint32_t i : by_cost) {
    const int home = static_cast<int>(i % kXcds);
    int any = -1;
    for (int x = 0; x < kXcds; ++x)
      if (!loads[x].empty() && (any < 0 || loads[x].top() < loads[any].top())) any = x;
    const double c = work_item_cost(items[i]);
    const int x = !loads[home].empty() && loads[home].top().first <= loads[any].top().first + 0.25 * c ? home : any;
    const Load least = loads[x].top();
    loads[x].pop();
    loads[x].push({least.first + c, least.second});
    owner[i] = least.second;
    ++first[least.second + 1];
  }
  for (int b = 0; b < grid; ++b) first[b + 1] += first[b];
  *ranges = first;
  std::vector<WorkItem> out(n_items);
  for (size_t i = 0; i < n_items; ++i) out[first[owner[i]]++] = items[i];
  std::copy(out.begin(), out.end(), items.begin());
}

std::vector<WorkItem> scheduled_list(const std::vector<WorkItem>& items, int grid, bool both,
                                     std::vector<uint32_t>* ranges) {
  ranges->clear();
  if (!needs_balance(items, grid)) return {};
  std::vector<WorkItem> balanced(items);
  balance_work_items(balanced, grid, ranges);
  if (!both) return balanced;
  std::vector<WorkItem> list;
  list.reserve(2 * items.size());
  list = items;
  list.insert(list.end(), balanced.begin(), balanced.end());
  return list;
}

void append_work_items(const cleave_task& t, uint32_t task_index, std::vector<WorkItem>* out,
                       bool fine) {
  const SubTiling s = sub_tiling(t, fine);
  for (uint32_t sub = 0; sub < s.count(); ++sub)
    out[s.cls].push_back(make_work_item(t, task_index, s, sub));
}

}  // namespace cleave

using cleave::Tile;

extern "C" int cleave_plan_uniform(int64_t M, int64_t N, int64_t K, int64_t tile_m, int64_t tile_n,
                                   int32_t ksplit, uint32_t gemm_id, cleave_plan** out) {
  if (!out) return CLEAVE_EINVAL;
  if (M < 1 || N < 1 || K < 1 || tile_m < 1 || tile_n < 1) return CLEAVE_EINVAL;
  if (M > cleave::kMaxDim || N > cleave::kMaxDim || K > cleave::kMaxDim) return CLEAVE_EINVAL;
  if (!cleave::valid_split(K, ksplit)) return CLEAVE_EINVAL;
  std::vector<Tile> tiles;
  try {
    for (int64_t m0 = 0; m0 < M; m0 += tile_m)
      for (int64_t n0 = 0; n0 < N; n0 += tile_n)
        tiles.push_back(Tile{m0, std::min(tile_m, M - m0), n0, std::min(tile_n, N - n0), ksplit});
  } catch (const std::bad_alloc&) {
    return CLEAVE_ENOMEM;
  }
  const int rc = cleave::finish_plan(M, N, K, tiles, gemm_id, out);
  if (rc == CLEAVE_OK) (*out)->uniform_splits = ksplit;
  return rc;
}

extern "C" int cleave_plan_batched(int64_t M, int64_t N, int64_t K, int64_t tile_m, int64_t tile_n,
                                   int32_t ksplit, int64_t n_batch, cleave_plan** out) {
  if (!out) return CLEAVE_EINVAL;
  if (M < 1 || N < 1 || K < 1 || tile_m < 1 || tile_n < 1 || n_batch < 1) return CLEAVE_EINVAL;
  if (M > cleave::kMaxDim || N > cleave::kMaxDim || K > cleave::kMaxDim ||
      n_batch > cleave::kMaxDim)
    return CLEAVE_EINVAL;
  if (!cleave::valid_split(K, ksplit)) return CLEAVE_EINVAL;
  std::vector<Tile> tiles;
  try {
    for (int64_t m0 = 0; m0 < M; m0 += tile_m)
      for (int64_t n0 = 0; n0 < N; n0 += tile_n)
        tiles.push_back(Tile{m0, std::min(tile_m, M - m0), n0, std::min(tile_n, N - n0), ksplit});
  } catch (const std::bad_alloc&) {
    return CLEAVE_ENOMEM;
  }
  return cleave::finish_plan(M, N, K, tiles, 0, out, n_batch);
}

extern "C" int cleave_plan_explicit(int64_t M, int64_t N, int64_t K, int32_t n_bands,
                                    const int64_t* band_h, const int32_t* n_cols,
                                    const int64_t* col_w, const int32_t* ksplit_per_tile,
                                    uint32_t gemm_id, cleave_plan** out) {
  if (!out || !band_h || !n_cols || !col_w || !ksplit_per_tile) return CLEAVE_EINVAL;
  if (M < 1 || N < 1 || K < 1 || n_bands < 1) return CLEAVE_EINVAL;
  if (M > cleave::kMaxDim || N > cleave::kMaxDim || K > cleave::kMaxDim) return CLEAVE_EINVAL;
  std::vector<Tile> tiles;
  try {
    int64_t m0 = 0;
    int64_t w_idx = 0;
    for (int32_t b = 0; b < n_bands; ++b) {
      const int64_t h = band_h[b];
      if (h < 1 || h > M - m0 || n_cols[b] < 1) return CLEAVE_EINVAL;
      int64_t n0 = 0;
      for (int32_t c = 0; c < n_cols[b]; ++c, ++w_idx) {
        const int64_t w = col_w[w_idx];
        if (w < 1 || w > N - n0) return CLEAVE_EINVAL;
        const int32_t S = ksplit_per_tile[tiles.size()];
        if (!cleave::valid_split(K, S)) return CLEAVE_EINVAL;
        tiles.push_back(Tile{m0, h, n0, w, S});
        n0 += w;
      }
      if (n0 != N) return CLEAVE_EINVAL;
      m0 += h;
    }
    if (m0 != M) return CLEAVE_EINVAL;
  } catch (const std::bad_alloc&) {
    return CLEAVE_ENOMEM;
  }
  return cleave::finish_plan(M, N, K, tiles, gemm_id, out);
}

extern "C" int64_t cleave_plan_num_tasks(const cleave_plan* plan) {
  return plan ? static_cast<int64_t>(plan->tasks.size()) : int64_t{CLEAVE_EINVAL};
}

extern "C" int64_t cleave_plan_num_tiles(const cleave_plan* plan) {
  return plan ? plan->num_tiles : int64_t{CLEAVE_EINVAL};
}

extern "C" const cleave_task* cleave_plan_tasks(const cleave_plan* plan) {
  return plan ? plan->tasks.data() : nullptr;
}

extern "C" int64_t cleave_plan_partial_elems(const cleave_plan* plan) {
  return plan ? plan->partial_elems : int64_t{CLEAVE_EINVAL};
}

extern "C" int cleave_plan_dims(const cleave_plan* plan, int64_t* dims) {
  if (!plan || !dims) return CLEAVE_EINVAL;
  dims[0] = plan->M;
  dims[1] = plan->N;
  dims[2] = plan->K;
  return CLEAVE_OK;
}

extern "C" const char* cleave_plan_last_kernel(const cleave_plan* plan) {
  return plan ? plan->last_kernel : "none";
}

extern "C" const char* cleave_strerror(int status) {
  switch (status) {
    case CLEAVE_OK: return "ok";
    case CLEAVE_EINVAL: return "invalid argument";
    case CLEAVE_ENOMEM: return "out of memory";
    case CLEAVE_EHIP: return "HIP runtime error";
    case CLEAVE_ELIMIT: return "request exceeds the fixed limit of this entry point";
    default: return "unknown status";
  }
}

extern "C" int cleave_plan_schedule_loads(const cleave_plan* plan, int list, int grid, int balanced,
                                          double* loads) {
  if (!plan || !loads || list < 0 || list > cleave::kNumTileClasses || grid < 1) return CLEAVE_EINVAL;
  const bool fine = list == cleave::kNumTileClasses;
  const std::vector<cleave::WorkItem>& host = fine ? plan->items_fine : plan->items[list];
  std::fill(loads, loads + grid, 0.0);
  try {
    std::vector<cleave::WorkItem> items(host);
    std::vector<uint32_t> ranges;
    if (balanced) cleave::balance_work_items(items, grid, &ranges);
    if (!ranges.empty()) {
      for (int b = 0; b < grid; ++b)
        for (uint32_t i = ranges[b]; i < ranges[b + 1]; ++i) loads[b] += cleave::work_item_cost(items[i]);
    } else {
      for (size_t i = 0; i < items.size(); ++i) loads[i % static_cast<size_t>(grid)] += cleave::work_item_cost(items[i]);
    }
  } catch (const std::bad_alloc&) {
    return CLEAVE_ENOMEM;
  }
  return CLEAVE_OK;
}
