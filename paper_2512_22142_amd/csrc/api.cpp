// C-ABI entry points that touch the device: table upload, execute, reduce.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <limits>
#include <map>
#include <mutex>
#include <new>
#include <utility>
#include <vector>

#include "kernels.h"
#include "plan_internal.h"

namespace {

thread_local int g_last_hip_error = 0;

int hip_fail(hipError_t e) {
  g_last_hip_error = static_cast<int>(e);
  return CLEAVE_EHIP;
}

#define CLEAVE_HIP(expr)                         \
  do {                                           \
    hipError_t e__ = (expr);                     \
    if (e__ != hipSuccess) return hip_fail(e__); \
  } while (0)

bool aligned(const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

void free_verify_device(cleave::VerifyTables* v) {
  if (!v) return;
  void* ptrs[] = {v->d_row_segs, v->d_col_segs, v->d_task_row_seg, v->d_task_col_seg,
                  v->d_items, v->d_task_first_item, v->d_agg_items, v->d_agg_first_item,
                  v->d_agg_item_sums, v->d_proj, v->d_item_sums};
  for (void* q : ptrs)
    if (q) (void)hipFree(q);
  v->d_row_segs = v->d_col_segs = nullptr;
  v->d_task_row_seg = v->d_task_col_seg = v->d_task_first_item = v->d_agg_first_item = nullptr;
  v->d_items = v->d_agg_items = nullptr;
  v->d_proj = v->d_item_sums = v->d_agg_item_sums = nullptr;
}

void free_subset_ring(cleave::SubsetRing* r) {
  if (r->d_ring) (void)hipFree(r->d_ring);
  if (r->d_captured) (void)hipFree(r->d_captured);
  for (const auto& f : r->in_flight) (void)hipEventDestroy(f.done);
  for (hipEvent_t e : r->idle_events) (void)hipEventDestroy(e);
  r->d_ring = r->d_captured = nullptr;
  r->in_flight.clear();
  r->idle_events.clear();
  r->max_items = r->pos = r->captured_used = 0;
}

void free_device_tables(cleave_plan* p) {
  free_verify_device(p->verify);
  if (p->d_tasks) (void)hipFree(p->d_tasks);
  for (int c = 0; c < cleave::kNumTileClasses; ++c)
    if (p->d_items[c]) (void)hipFree(p->d_items[c]);
  if (p->d_reduce_items) (void)hipFree(p->d_reduce_items);
  free_subset_ring(&p->subset);
  p->d_tasks = nullptr;
  if (p->d_items_fine) (void)hipFree(p->d_items_fine);
  p->d_items_fine = nullptr;
  for (int list = 0; list < cleave::kNumTileClasses + 1; ++list) {
    if (p->d_wg_ranges[list]) (void)hipFree(p->d_wg_ranges[list]);
    p->d_wg_ranges[list] = nullptr;
    p->wg_ranges_grid[list] = 0;
  }
  p->d_items[0] = p->d_items[1] = nullptr;
  p->d_reduce_items = nullptr;
  p->device = -1;
}

template <typename T>
int upload_vector(const std::vector<T>& v, T** dst) {
  *dst = nullptr;
  if (v.empty()) return CLEAVE_OK;
  hipError_t e = hipMalloc(reinterpret_cast<void**>(dst), v.size() * sizeof(T));
  if (e == hipErrorOutOfMemory) return CLEAVE_ENOMEM;
  if (e != hipSuccess) return hip_fail(e);
  CLEAVE_HIP(hipMemcpy(*dst, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice));
  return CLEAVE_OK;
}

// The current device's stream for kernels of an upload: made by the first upload
// that needs it, held until the process ends.
constexpr int kMaxDevices = 64;
std::mutex g_upload_mu;
hipStream_t g_upload_stream[kMaxDevices] = {};
int upload_stream(hipStream_t* out) {
  int dev = 0;
  CLEAVE_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return CLEAVE_EINVAL;
  std::lock_guard<std::mutex> lock(g_upload_mu);
  if (!g_upload_stream[dev]) CLEAVE_HIP(hipStreamCreateWithFlags(&g_upload_stream[dev], hipStreamNonBlocking));
  *out = g_upload_stream[dev];
  return CLEAVE_OK;
}

// The aggregation's table, from the tasks already on the device and the tile list
// (which goes behind the records).  The kernel that writes it is on the device's
// own upload stream, so that neither it nor the caller's wait for it stands
// behind work that the program has on the null stream (on that stream, preparing
// three plans of 16384 x 13824 beside their operands took 12.7 ms, 10.5 without),
// and the caller waits behind its other uploads, which overlap it.  A short table
// is written by the host and copied (2 ns a record; launch and wait cost 25 us).
constexpr int64_t kHostRecords = 8192;
int make_reduce_table(cleave_plan* p, hipStream_t* used) {
  *used = nullptr;
  if (p->reduce_runs <= kHostRecords) {
    try {
      std::vector<cleave::ReduceItem> records;
      records.reserve(static_cast<size_t>(p->reduce_runs));
      for (const cleave::ReduceTile& tile : p->reduce_tiles) {
        const cleave_task& t = p->tasks[tile.task];
        const uint64_t block = static_cast<uint64_t>(t.m_len) * t.n_len;
        for (uint64_t e = 0; e < block; e += tile.run) records.push_back(cleave::make_reduce_item(t, e, tile.run));
      }
      return upload_vector(records, &p->d_reduce_items);
    } catch (const std::bad_alloc&) {
      return CLEAVE_ENOMEM;
    }
  }
  const int64_t n_tiles = static_cast<int64_t>(p->reduce_tiles.size());
  const size_t records = static_cast<size_t>(p->reduce_runs) * sizeof(cleave::ReduceItem);
  const size_t listed = p->reduce_tiles.size() * sizeof(cleave::ReduceTile);
  unsigned char* table = nullptr;
  const hipError_t e = hipMalloc(reinterpret_cast<void**>(&table), records + listed);
  if (e == hipErrorOutOfMemory) return CLEAVE_ENOMEM;
  if (e != hipSuccess) return hip_fail(e);
  p->d_reduce_items = reinterpret_cast<cleave::ReduceItem*>(table);
  cleave::ReduceTile* tiles = reinterpret_cast<cleave::ReduceTile*>(table + records);
  CLEAVE_HIP(hipMemcpy(tiles, p->reduce_tiles.data(), listed, hipMemcpyHostToDevice));
  hipStream_t stream = nullptr;
  const int rc = upload_stream(&stream);
  if (rc != CLEAVE_OK) return rc;
  CLEAVE_HIP(cleave::launch_expand_reduce(p->d_tasks, tiles, n_tiles, p->d_reduce_items, stream));
  *used = stream;
  return CLEAVE_OK;
}

// Work-list memory of cleave_execute_noalloc: a fixed array in the code
// object, one copy per GPU the library runs on, held until the process ends
// (768 KB).  In host code the name is only a handle for hipGetSymbolAddress;
// the address that kernels and copies use is g_static_scratch[device].
constexpr int64_t kStaticScratchItems = 16384;
static __device__ __align__(256) __attribute__((used))
unsigned char scratch[kStaticScratchItems * sizeof(cleave::WorkItem)];

// Once per device and process: the execute kernels' dynamic-LDS limits, the
// CU count and the address of this device's copy of `scratch`.  Done when a
// plan's tables are uploaded, so that no launch has to.
std::mutex g_device_mu;
int g_device_cus[kMaxDevices] = {};   // 0 = not initialised
cleave::WorkItem* g_static_scratch[kMaxDevices] = {};

int ensure_device_ready(int dev, int* cus) {
  if (dev < 0 || dev >= kMaxDevices) return CLEAVE_EINVAL;
  std::lock_guard<std::mutex> lock(g_device_mu);
  if (g_device_cus[dev] == 0) {
    CLEAVE_HIP(cleave::configure_execute_kernels());
    CLEAVE_HIP(cleave::configure_execute_direct_kernels());
    void* ptr = nullptr;   // `dev` is the current device: its copy of the array
    CLEAVE_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    g_static_scratch[dev] = static_cast<cleave::WorkItem*>(ptr);
    int n = 0;
    CLEAVE_HIP(hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev));
    g_device_cus[dev] = std::max(n, 1);
  }
  if (cus) *cus = g_device_cus[dev];
  return CLEAVE_OK;
}

constexpr int kSubsetEvents = 16;

int allocate_subset_ring(cleave_plan* p) {
  cleave::SubsetRing& r = p->subset;
  r.max_items = static_cast<int64_t>(std::max(p->items[0].size() + p->items[1].size(), p->items_fine.size()));
  if (r.max_items == 0) return CLEAVE_OK;
  const size_t item_bytes = static_cast<size_t>(r.max_items) * sizeof(cleave::WorkItem);
  hipError_t e = hipMalloc(reinterpret_cast<void**>(&r.d_ring), 2 * item_bytes);
  if (e == hipSuccess) e = hipMalloc(reinterpret_cast<void**>(&r.d_captured), item_bytes);
  if (e == hipErrorOutOfMemory) return CLEAVE_ENOMEM;
  if (e != hipSuccess) return hip_fail(e);
  try {
    r.idle_events.reserve(kSubsetEvents);
    r.in_flight.reserve(kSubsetEvents);
  } catch (const std::bad_alloc&) {
    return CLEAVE_ENOMEM;
  }
  for (int i = 0; i < kSubsetEvents; ++i) {
    hipEvent_t ev = nullptr;
    CLEAVE_HIP(hipEventCreateWithFlags(&ev, hipEventDisableTiming));
    r.idle_events.push_back(ev);
  }
  return CLEAVE_OK;
}

bool cut_small(const cleave_plan* plan, int cus);

int ensure_uploaded(cleave_plan* p) {
  int dev = 0;
  CLEAVE_HIP(hipGetDevice(&dev));
  if (p->device == dev) return CLEAVE_OK;
  if (p->device >= 0) free_device_tables(p);
  int rc = ensure_device_ready(dev, nullptr);
  if (rc != CLEAVE_OK) return rc;
  rc = upload_vector(p->tasks, &p->d_tasks);
  hipStream_t writing = nullptr;
  if (rc == CLEAVE_OK) rc = make_reduce_table(p, &writing);
  // The three work-item lists; items of unequal length get a balanced workgroup
  // schedule for this device's grid (the host lists keep their canonical order for
  // the next device).  Full launches of the general kernel run the third list, the
  // fast kernel's only where it cuts large blocks small.
  int cus = 0;
  if (rc == CLEAVE_OK) rc = ensure_device_ready(dev, &cus);
  for (int list = 0; rc == CLEAVE_OK && list < cleave::kNumTileClasses + 1; ++list) {
    const bool fine = list == cleave::kNumTileClasses;
    const int cls = fine ? cleave::kTileSmall : list;
    const std::vector<cleave::WorkItem>& host = fine ? p->items_fine : p->items[list];
    cleave::WorkItem** dst = fine ? &p->d_items_fine : &p->d_items[list];
    const int64_t resident = static_cast<int64_t>(cus) * cleave::direct_workgroups_per_cu(
                                                                cls == cleave::kTileLarge ? cleave::kDirectLarge : cleave::kDirectSmall);
    const int grid = static_cast<int>(std::min<int64_t>(static_cast<int64_t>(host.size()), resident));
    std::vector<uint32_t> ranges;
    try {
      std::vector<cleave::WorkItem> scheduled;
      if (!fine || cut_small(p, cus)) scheduled = cleave::scheduled_list(host, grid, fine, &ranges);
      rc = upload_vector(ranges.empty() ? host : scheduled, dst);
    } catch (const std::bad_alloc&) {
      rc = CLEAVE_ENOMEM;
    }
    if (rc == CLEAVE_OK && !ranges.empty()) {
      rc = upload_vector(ranges, &p->d_wg_ranges[list]);
      p->wg_ranges_grid[list] = grid;
    }
  }
  if (rc == CLEAVE_OK) rc = allocate_subset_ring(p);
  if (writing) {   // the tables are read on any stream next (and freed on an error)
    const hipError_t e = hipStreamSynchronize(writing);
    if (e != hipSuccess && rc == CLEAVE_OK) rc = hip_fail(e);
  }
  if (rc != CLEAVE_OK) {
    free_device_tables(p);
    return rc;
  }
  p->device = dev;
  return CLEAVE_OK;
}

int compute_units(int* out) {
  int dev = 0;
  CLEAVE_HIP(hipGetDevice(&dev));
  return ensure_device_ready(dev, out);
}

// A slice of `total` work items for a subset launch on `stream`.  Eager
// launches take the next slice of the ring (waiting, on the host, only for
// earlier launches that still read the slice: none unless the ring has
// wrapped onto unfinished work); launches under stream capture take a slice
// of the second buffer that is never handed out again.  No allocation.
int acquire_subset_slice(cleave::SubsetRing& r, int64_t total, bool capturing, cleave::WorkItem** out,
                         int64_t* begin) {
  if (total > r.max_items) return CLEAVE_EINVAL;   // cannot happen for distinct task ids
  if (capturing) {
    if (r.captured_used + total > r.max_items) return CLEAVE_ENOMEM;
    *out = r.d_captured + r.captured_used;
    *begin = -1;
    r.captured_used += total;
    return CLEAVE_OK;
  }
  if (r.pos + total > 2 * r.max_items) r.pos = 0;
  const int64_t b = r.pos, e = r.pos + total;
  // launches retire in order per stream, not across streams: check every record
  for (size_t i = 0; i < r.in_flight.size();) {
    const auto f = r.in_flight[i];
    const bool overlaps = f.begin < e && b < f.end;
    hipError_t q = overlaps ? hipEventSynchronize(f.done) : hipEventQuery(f.done);
    if (q == hipSuccess) {
      r.idle_events.push_back(f.done);
      r.in_flight.erase(r.in_flight.begin() + static_cast<std::ptrdiff_t>(i));
    } else if (q == hipErrorNotReady) {
      ++i;
    } else {
      return hip_fail(q);
    }
  }
  *out = r.d_ring + b;
  *begin = b;
  r.pos = e;
  return CLEAVE_OK;
}

// Marks the slice [begin, begin + total) as read by what has been enqueued on
// `stream` so far.
int release_subset_slice(cleave::SubsetRing& r, int64_t begin, int64_t total, hipStream_t stream) {
  if (begin < 0) return CLEAVE_OK;   // captured: never reused
  if (r.idle_events.empty()) {
    // every event is attached to a launch still in flight: wait for the oldest
    const auto f = r.in_flight.front();
    CLEAVE_HIP(hipEventSynchronize(f.done));
    r.in_flight.erase(r.in_flight.begin());
    r.idle_events.push_back(f.done);
  }
  hipEvent_t ev = r.idle_events.back();
  r.idle_events.pop_back();
  const hipError_t e = hipEventRecord(ev, stream);
  if (e != hipSuccess) {
    r.idle_events.push_back(ev);
    return hip_fail(e);
  }
  r.in_flight.push_back({begin, begin + total, ev});
  return CLEAVE_OK;
}

const char* kernel_name(int dtype, const cleave::GeneralLoads& how, int transA, int transB) {
  static const char* names[2][6][4] = {
      {{"execute_f32_128x128_nn", "execute_f32_128x128_nt", "execute_f32_128x128_tn", "execute_f32_128x128_tt"},
       {"execute_f32_64x64_nn", "execute_f32_64x64_nt", "execute_f32_64x64_tn", "execute_f32_64x64_tt"},
       {"none", "none", "none", "none"},
       {"execute_f32_64x64_quarters_nn", "execute_f32_64x64_quarters_nt", "execute_f32_64x64_quarters_tn",
        "execute_f32_64x64_quarters_tt"},
       {"execute_f32_element", "execute_f32_element", "execute_f32_element", "execute_f32_element"},
       {"execute_f32_64x64_lone_nn", "execute_f32_64x64_lone_nt", "execute_f32_64x64_lone_tn", "execute_f32_64x64_lone_tt"}},
      {{"execute_bf16_128x128_nn", "execute_bf16_128x128_nt", "execute_bf16_128x128_tn", "execute_bf16_128x128_tt"},
       {"execute_bf16_64x64_nn", "execute_bf16_64x64_nt", "execute_bf16_64x64_tn", "execute_bf16_64x64_tt"},
       {"none", "execute_bf16_256x256_nt", "none", "none"},
       {"none", "none", "none", "none"},
       {"execute_bf16_element", "execute_bf16_element", "execute_bf16_element", "execute_bf16_element"},
       {"execute_bf16_64x64_lone_nn", "execute_bf16_64x64_lone_nt", "execute_bf16_64x64_lone_tn",
        "execute_bf16_64x64_lone_tt"}}};
  const int row = how.a_elements || how.b_elements ? 4 : how.tile == cleave::kTileWide4 ? cleave::kTileWide : how.tile;
  return names[dtype == CLEAVE_BF16 ? 1 : 0][row][(transA ? 2 : 0) + (transB ? 1 : 0)];
}

const char* direct_kernel_name(cleave::DirectShape shape, int transA, int transB) {
  static const char* names[4][4] = {
      {"execute_direct_bf16_256x256_nn", "execute_direct_bf16_256x256_nt",
       "execute_direct_bf16_256x256_tn", "execute_direct_bf16_256x256_tt"},
      {"execute_direct_bf16_128x128_nn", "execute_direct_bf16_128x128_nt",
       "execute_direct_bf16_128x128_tn", "execute_direct_bf16_128x128_tt"},
      {"execute_direct_bf16_128x128_deep_nn", "execute_direct_bf16_128x128_deep_nt",
       "execute_direct_bf16_128x128_deep_tn", "execute_direct_bf16_128x128_deep_tt"},
      {"execute_direct_bf16_64x64_nn", "execute_direct_bf16_64x64_nt",
       "execute_direct_bf16_64x64_tn", "execute_direct_bf16_64x64_tt"}};
  return names[shape][(transA ? 2 : 0) + (transB ? 1 : 0)];
}

}  // namespace

extern "C" int cleave_last_hip_error(void) { return g_last_hip_error; }

extern "C" int cleave_version(void) { return 107; }

extern "C" int cleave_plan_upload(cleave_plan* plan) {
  if (!plan) return CLEAVE_EINVAL;
  return ensure_uploaded(plan);
}

extern "C" void cleave_plan_destroy(cleave_plan* plan) {
  if (!plan) return;
  if (plan->device >= 0) free_device_tables(plan);
  delete plan->verify;
  delete plan;
}

namespace {

// How a batched call finds its members' matrices (element offsets from the
// base pointers); all zero for a plain plan.
struct BatchLayout {
  cleave::BatchShape shape{0, 0};
  cleave::MemberOffsets a{}, b{};
  cleave::MemberOffsets c{};   // assemble mode and reduce only
};

// Every member offset is a multiple of `e` elements.
bool offsets_multiple_of(const cleave::MemberOffsets& at, const cleave::BatchShape& shape, int64_t e) {
  if (shape.n_group == 0) return at.outer % e == 0 && at.inner % e == 0;
  for (uint32_t g = 0; g < shape.n_group; ++g)
    if (at.table[g] % e != 0) return false;
  return true;
}

BatchLayout strided_layout(int64_t n_inner, int64_t a_outer, int64_t a_inner, int64_t b_outer,
                           int64_t b_inner, int64_t c_outer, int64_t c_inner) {
  BatchLayout bl;
  bl.shape.batch_inner = static_cast<uint32_t>(n_inner);
  bl.a.outer = a_outer;
  bl.a.inner = a_inner;
  bl.b.outer = b_outer;
  bl.b.inner = b_inner;
  bl.c.outer = c_outer;
  bl.c.inner = c_inner;
  return bl;
}

// Grouped launch: members given by one pointer each.  list[0] becomes the base
// pointer, the others element offsets from it.
int group_offsets(const void* const* list, int64_t n, int elem_bytes, cleave::MemberOffsets* at,
                  const void** base) {
  if (!list || n < 1 || n > cleave::kMaxGroup) return CLEAVE_EINVAL;
  for (int64_t g = 0; g < n; ++g)
    if (!list[g] || !aligned(list[g], elem_bytes)) return CLEAVE_EINVAL;
  *base = list[0];
  for (int64_t g = 0; g < n; ++g)
    at->table[g] = (reinterpret_cast<intptr_t>(list[g]) - reinterpret_cast<intptr_t>(list[0])) / elem_bytes;
  return CLEAVE_OK;
}

// Assemble mode: blocks go to their place in C instead of the partial buffer.
struct AssembleTarget {
  void* C = nullptr;
  int64_t ldc = 0;
  int out_dtype = CLEAVE_F32;
};

// The work items of a full launch whose chunk starts below the returned k leave
// through non-temporal stores.  An output that the cache cannot hold pushes its own
// first part (and the operands) out of it, and the next launch waits for those
// write-backs; a streamed one goes to memory without them.  One that it can hold is
// read from there by whoever comes next.
//   Assembled outputs: see streamed_output.
//   Partial blocks of uniform plans (their items run chunk by chunk): execute +
// reduce over plain, all chunks but the last streamed / all of them streamed:
//   blocks of a chunk x chunks
//    67 MB x 4   1.031, 0.998 / 1.043, 1.005      67 MB x 8   0.893, 0.894 / 0.907, 0.901
//   134 MB x 2   1.034, 0.992 / 1.033, 0.991     134 MB x 4   0.884, 0.927 / 0.904, 0.920
//   134 MB x 8   0.911, 0.975 / 0.862, 0.992     180 MB x 2   0.969, 0.955 / 0.979, 0.954
//   180 MB x 4   0.945, 0.980 / 0.925, 0.965     180 MB x 8   0.984, 0.978 / 0.922, 0.988
//   268 MB x 4   1.001, 0.986 / 0.921, 1.005     268 MB x 8   0.968, 0.984 / 0.988, 0.981
//   336 MB x 2   0.976, 0.985 / 1.029, 1.002     336 MB x 8   0.955, 0.974 / 0.959, 0.967
//   453 MB x 2   0.989, 0.991 / 1.012, 0.996     453 MB x 4   0.967, 0.980 / 0.971, 0.980
//   453 MB x 8   0.981 / 0.971                   537 MB x 2   1.011, 1.007 / 1.025, 1.015
//   537 MB x 4   0.977, 0.989 / 0.974, 0.982     537 MB x 8   0.972 / 0.958
//   906 MB x 2   0.985, 0.991 / 0.970, 0.981     906 MB x 8   0.891 / 0.879
// (chunks of 512 and of 1024 elements, 1024 alone where one figure is given).  537 MB x 2
// (8192 x 16384) loses 1 % in every form, again in a second run (1.016, 1.010); beside it
// 528 MB x 2 0.998, 1.011, 604 MB x 2 0.985, 0.993, so no line by size leaves it out.
// Batched, grouped and explicit plans have not been measured and keep plain stores.  Short
// chains, whose launches are bound by the stores themselves, lose: linear layers, us,
// plain / streamed, chunks of 48 elements 292 / 302, of 63 494 / 512, of 82 525 / 531, of
// 200 639 / 651; of 476 1703 / 1612.
uint32_t streamed_below(const cleave_plan* plan, const AssembleTarget& asm_to) {
  const int64_t members = std::max<int64_t>(plan->batch, 1);
  const int64_t outputs = plan->M * plan->N * members;
  if (asm_to.C) {
    const int64_t bytes = outputs * (asm_to.out_dtype == CLEAVE_BF16 ? 2 : 4);
    return cleave::streamed_output(bytes, plan->batch > 0) ? static_cast<uint32_t>(plan->K) : 0;
  }
  const int64_t splits = plan->uniform_splits;
  if (splits < 2 || 4 * plan->partial_elems < cleave::kCacheBytes / 4 * 5) return 0;
  const int64_t chunk = (plan->K + splits - 1) / splits;
  if (chunk < 6 * int64_t{cleave::kDirectKStep}) return 0;
  const bool all = 4 * outputs >= 3 * cleave::kCacheBytes || (4 * outputs >= cleave::kCacheBytes / 2 * 3 && splits >= 4);
  return static_cast<uint32_t>(all ? plan->K : (splits - 1) * chunk);
}

// Where the work items of a subset go: one list per tile class, in the caller's
// order (the layout of the plan's own lists).
struct SubsetLayout {
  bool fine = false;                               // every block cut into small-class sub-tiles
  int64_t counts[cleave::kNumTileClasses] = {};    // work items per class
  int64_t steps[cleave::kNumTileClasses] = {};     // their whole K steps, together
  cleave::ListShape shapes[cleave::kNumTileClasses];
  int64_t total() const { return counts[0] + counts[1]; }
};

// Validates the ids (range, no repeats) and sizes the lists.  Uses the plan's
// own stamp array for the repeat check: no allocation.  Caller holds subset.mu.
// The cut depends on the ids alone, not on which kernel runs the items (the
// general one cuts large items into its workgroup tiles itself), so neither do
// the work-list memory a subset takes and the limit on it.
int layout_subset(cleave_plan* plan, const int64_t* task_ids, int64_t n_ids, int cus, SubsetLayout* out) {
  const int64_t n_tasks = static_cast<int64_t>(plan->tasks.size());
  if (++plan->seen_generation == 0) {   // wrapped: start over with clean stamps
    std::fill(plan->seen_stamp.begin(), plan->seen_stamp.end(), 0u);
    plan->seen_generation = 1;
  }
  size_t large_items = 0;
  for (int64_t i = 0; i < n_ids; ++i) {
    const int64_t id = task_ids[i];
    if (id < 0 || id >= n_tasks || plan->seen_stamp[id] == plan->seen_generation) return CLEAVE_EINVAL;
    plan->seen_stamp[id] = plan->seen_generation;
    const cleave::SubTiling st = cleave::sub_tiling(plan->tasks[id], false);
    if (st.cls == cleave::kTileLarge) large_items += st.count();
  }
  // Few large items would leave most CUs idle: cut everything small instead
  // (the bits do not depend on the cut).
  out->fine = large_items > 0 && large_items <= static_cast<size_t>(cus) / 2;
  for (int64_t i = 0; i < n_ids; ++i) {
    const cleave_task& t = plan->tasks[task_ids[i]];
    const cleave::SubTiling st = cleave::sub_tiling(t, out->fine);
    out->counts[st.cls] += st.count();
    out->steps[st.cls] += int64_t{st.count()} * (t.k_len / cleave::kDirectKStep);
    out->shapes[st.cls].add(t);
  }
  return CLEAVE_OK;
}

// Enqueues the kernels that write the subset's work items to `out`; the
// (task, destination) pairs are built on the stack, one launch's worth at a time.
int expand_subset(const cleave_plan* plan, const int64_t* task_ids, int64_t n_ids,
                  const SubsetLayout& layout, cleave::WorkItem* out, hipStream_t stream) {
  int64_t next[cleave::kNumTileClasses] = {0, layout.counts[0]};
  cleave::ExpandArgs ea{};
  ea.tasks = plan->d_tasks;
  ea.out = out;
  ea.fine = layout.fine ? 1u : 0u;
  for (int64_t i = 0; i < n_ids; ++i) {
    const cleave_task& t = plan->tasks[task_ids[i]];
    const cleave::SubTiling st = cleave::sub_tiling(t, layout.fine);
    int64_t& at = next[st.cls];
    ea.entries[ea.n_entries++] = {static_cast<uint32_t>(task_ids[i]), static_cast<uint32_t>(at)};
    at += st.count();
    if (ea.n_entries == cleave::kSubsetEntriesPerLaunch || i + 1 == n_ids) {
      CLEAVE_HIP(cleave::launch_expand_subset(ea, stream));
      ea.n_entries = 0;
    }
  }
  return CLEAVE_OK;
}

// Workgroup tile of the general kernel for `items` 128 x 128 work items.  The
// 64 x 64 tile gives four times as many workgroups, four of them per CU
// instead of two, at twice the LDS traffic per flop.  fp32 MFMAs leave the LDS
// mostly idle, so there the narrow tile wins unless the wide one's workgroups fill
// their rounds of the CUs to 15/16 (from four rounds on it runs whether or not).  us, wide /
// narrow, layouts NN, NT, TN: 32 steps, 256 items 71 / 68, 70 / 67, 72 / 69, 480 items
// 125 / 129, 123 / 127, 127 / 129, 704 items 183 / 182, 184 / 177, 183 / 183, 768 items 184 /
// 196, 185 / 191, 184 / 195, 896 items 246 / 227, 242 / 226, 249 / 229; 12 steps, 480 items
// 52.7 / 54.1, 52.3 / 54.0, 53.5 / 55.1, 768 items 76.4 / 81.2, 76.3 / 81.9, 77.4 / 80.9.
// The wide tile multiplies all of an item, the narrow one the 64 x 64 parts that hold
// something (`list.parts64` in all): with small blocks there is less to win.  Below four
// rounds it runs from four fifths on, from there on from a half.  fp32, 1024 of K, by what
// the items hold: 960 items 0.56 246 / 230, 242 / 225, 248 / 231; 720 items 0.88 183 / 186,
// 184 / 183, 183 / 187; 512 items of 64 x 64 blocks (0.25, 512 of K) 64 / 22, 64 / 21, 66 / 22;
// 1024 items 0.25 244 / 68, 241 / 67, 248 / 68, 0.52 246 / 246, 242 / 241, 248 / 246; 2048 items
// 0.5 252 / 136, 251 / 134, 255 / 135; 2560 items 0.56 314 / 316, 314 / 308, 318 / 318, with 256
// of K 97 / 102, 97 / 102, 100 / 106.
// bf16 MFMAs do not: narrow only while the wide tile leaves half of the CUs without a
// workgroup (11 steps, 128 items 14.6 / 12.6, 13.7 / 12.4, 14.5 / 12.4, 192 items 15.2 /
// 17.4, 15.1 / 17.7, 15.5 / 17.4; 3 to 6 steps, 64 items 9.6 / 7.1, 192 items 9.5 / 10.0).
// Few fp32 items run as quarters of the 64 x 64 tile, up to two on each CU: a wave's
// chain of matrix instructions is what such a launch takes, and a quarter's is a
// quarter as long (with four times the waves, half as many products per load).
// Execute alone, us, 64 x 64 / quarters, operands in L2, layouts NN, NT, TN, TT (64 x 64 as it
// runs: the form that reads ahead from eight steps on): 16 items of 32 of K 4.0 / 3.9, 3.8 / 3.8,
// 4.1 / 3.8, 4.1 / 3.9, of 128 5.9 / 4.8, 5.7 / 4.9, 6.0 / 4.4, 6.0 / 4.8, of 512 12.4 / 8.1, 12.2 / 8.6,
// 12.5 / 7.0, 12.2 / 8.1, of 2048 37 / 20.9, 37 / 22.9, 37 / 17.2, 37 / 21.2; 32 items of 32 4.1 / 4.4,
// 3.9 / 4.4, 4.3 / 4.2, 4.2 / 4.4, of 64 4.8 / 4.7, 4.6 / 4.7, 4.9 / 4.5, 4.8 / 4.7, of 96 5.5 / 5.3,
// 5.2 / 5.3, 5.6 / 5.0, 5.5 / 5.1, of 128 6.1 / 5.7, 5.9 / 5.9, 6.2 / 5.3, 6.1 / 5.6, of 160 6.8 / 6.1,
// 6.6 / 6.4, 6.9 / 5.7, 6.8 / 6.1, of 256 8.4 / 7.3, 8.2 / 7.7, 8.6 / 6.6, 8.3 / 7.3, of 1024 20.9 / 16.6,
// 20.8 / 19.0, 21.0 / 14.3, 20.8 / 17.0 (20 and 24 items as 32); 40 items of 256 8.5 / 8.6, 8.3 / 9.5,
// 8.7 / 7.9, 8.4 / 8.6, of 1024 21.0 / 21.2, 21.0 / 24.3, 21.3 / 19.1, 21.0 / 21.8; 64 of 512 13.1 / 15.5,
// 13.0 / 17.4, 13.2 / 13.9, 13.1 / 15.6.  With two on a CU, beyond 16 items, only chunks from 128
// elements on, of two K-contiguous operands (whose fragments take twice the reads) from 256.  That
// is on the safe side: the lines were drawn on forms of both that read nothing ahead, and below them the
// quarters now gain too, from 160 on in NT, from 64 on in NN and TT (1 to 6 %), at any length in TN (2 to 15 %).
// `whole`: that many 256 x 256 items of a subset (full launches of this kernel run
// the all-small list), with `steps` whole K steps between them, that the kernel
// could take as they are (bf16, both operands K-contiguous: six
// fragment reads for eight products instead of eight).  They win when their
// rounds are nearly full and their chains long enough to cover a start and end
// alone on a CU (us, 128 / 256: 17 steps, 256 items 57 / 50, 1024 items 230 / 193, 688 items 144 / 132,
// 576 items, the third round a quarter full, 116 / 127; 5 steps, 1024 items
// 92.7 / 92.6, 688 items 59 / 66).
cleave::ExecuteTile general_tile(int dtype, bool both_k, int64_t items, const cleave::ListShape& list, int64_t whole,
                                 int64_t steps, int cus) {
  const int64_t places = (whole + cus - 1) / cus * cus;
  if (whole > 0 && whole * 8 >= places * 7 && steps >= 16 * whole) return cleave::kTileHuge;
  if (dtype == CLEAVE_F32 && 8 * items <= cus && (16 * items <= cus || list.longest >= (both_k ? 256u : 128u)))
    return cleave::kTileQuarter;
  if (dtype == CLEAVE_BF16) return 2 * items <= cus ? cleave::kTileNarrow : cleave::kTileWide;
  const int64_t places_wide = (items + cus - 1) / cus * cus;
  const bool wide = items >= int64_t{4} * cus
                        ? list.parts64 > 2 * items
                        : items > cus && 16 * items >= 15 * places_wide && 5 * list.parts64 >= 16 * items;
  return wide ? cleave::kTileWide : cleave::kTileNarrow;
}

// Shape of the direct kernel for `items` work items of a class.  Small items run as 64 x 64
// parts while a part has a place of its own, two on each CU (an item is four of them): there
// parts win at every chain length.  From there to one item per CU the deep ring does.  Time
// against 128 x 128 items with two stages, operands in L2 / from HBM, the largest of three
// layouts, by K steps per item (256 CUs):
//                    2 steps      4            8            16           24           48
//    16 items parts  0.65 / 0.65  0.63 / 0.63  0.60 / 0.60  0.57 / 0.51  0.56 / 0.45  0.54 / 0.42
//             deep   0.85 / 0.85  0.88 / 0.88  0.91 / 0.88  0.94 / 0.81  0.95 / 0.75  0.98 / 0.75
//    64 items parts  0.70 / 0.70  0.67 / 0.67  0.64 / 0.62  0.61 / 0.56  0.59 / 0.53  0.49 / 0.48
//             deep   0.87 / 0.86  0.89 / 0.88  0.92 / 0.86  0.94 / 0.83  0.96 / 0.83  0.81 / 0.79
//   128 items parts  0.78 / 0.78  0.78 / 0.79  0.79 / 0.80  0.77 / 0.79  0.78 / 0.78  0.77 / 0.78
//             deep   0.88 / 0.86  0.89 / 0.91  0.92 / 0.88  0.94 / 0.85  0.95 / 0.84  0.80 / 0.81
//   130 items parts  0.92 / 0.95  0.94 / 0.94  0.98 / 0.93  1.01 / 0.88  0.88 / 0.89  0.86 / 0.81
//             deep   0.88 / 0.87  0.91 / 0.91  0.92 / 0.86  0.93 / 0.80  0.78 / 0.78  0.72 / 0.72
//   160 items parts  0.97 / 0.98  0.98 / 0.98  1.02 / 0.98  0.98 / 0.91  0.96 / 0.92  0.95 / 0.93
//             deep   0.88 / 0.88  0.91 / 0.90  0.92 / 0.87  0.93 / 0.83  0.90 / 0.76  0.78 / 0.73
//   224 items deep   0.89 / 0.89  0.92 / 0.91  0.92 / 0.88  0.93 / 0.82  0.83 / 0.76  0.83 / 0.74
//   256 items deep   0.90 / 0.90  0.92 / 0.92  0.93 / 0.87  0.91 / 0.80  0.83 / 0.76  0.85 / 0.73
// (Before its last steps were copies with constant waits the ring took 1.09 to 1.14 of the two-stage time
// with operands in L2 at 4 and 8 steps, and ran from 16 on only.)  Two such launches at a time, on
// two streams, 4 to 24 steps: deep 0.87 to 0.98 of two stages with 136 or 160 items each, 0.95 to 1.02
// with 192, 1.11 to 1.17 with 256, when a CU would have held a two-stage workgroup of each.
cleave::DirectShape direct_shape(int cls, int64_t items, int cus) {
  if (cls == cleave::kTileLarge) return cleave::kDirectLarge;
  if (items * 2 <= cus) return cleave::kDirectParts;
  return items <= cus ? cleave::kDirectDeep : cleave::kDirectSmall;
}

// Whether a full launch of the direct kernel cuts every block into small sub-tiles:
// four times as many items, two workgroups per CU.  They cost more per product
// (twice the operand traffic into LDS, 1.1-1.25 times the time from four full
// rounds on), but a round is a quarter as much work, so they win where large items
// leave much of the last round's CUs idle.  The bits do not depend on the cut.
// Time of the small cut over the large one's, operands and blocks as the launch
// before left them in the caches / not in any cache (256 CUs, items of equal
// length; of three layouts and of square outputs and ones 1024 wide, where cold
// operands cost the small cut most, the one with the largest product of the two):
//            2 steps      4            8            12           16           24
//   136      0.88 / 0.89  0.94 / 1.00  0.98 / 1.08  1.01 / 1.14  1.02 / 1.19  1.07 / 1.25
//   192      0.91 / 0.92  0.89 / 0.98  0.95 / 1.07  0.96 / 1.18  0.96 / 1.20  0.97 / 1.33
//   224      0.98 / 0.97  0.93 / 1.12  0.97 / 1.33  1.01 / 1.45  1.04 / 1.48  1.05 / 1.51
//   272      0.81 / 0.94  0.74 / 1.06  0.75 / 1.10  0.78 / 1.11  0.78 / 1.12  0.80 / 1.13
//   288      0.81 / 0.94  0.75 / 1.09  0.76 / 1.11  0.78 / 1.15  0.80 / 1.13  0.82 / 1.16
//   320      0.86 / 0.97  0.84 / 1.02  0.81 / 1.04  0.79 / 1.12  0.81 / 1.13  0.81 / 1.15
//   352      0.92 / 1.09  0.90 / 1.19  0.87 / 1.21  0.88 / 1.25  0.90 / 1.21  0.90 / 1.23
//   384      0.89 / 1.05  0.93 / 1.16  0.89 / 1.25  0.90 / 1.24  0.92 / 1.23  0.91 / 1.25
//   544      0.89 / 1.01  0.83 / 1.13  0.88 / 1.12  0.86 / 1.21  0.86 / 1.18  0.85 / 1.21
//   576      0.89 / 1.05  0.84 / 1.14  0.88 / 1.22  0.91 / 1.24  0.89 / 1.23  1.04 / 1.30
//   640      0.92 / 1.18  0.93 / 1.22  0.94 / 1.32  0.96 / 1.33  0.95 / 1.25  1.23 / 1.33
// Chains of 64 steps: 272 items 0.87 / 0.94, 288 0.87 / 1.02.  Where some blocks are
// small anyway (a rim of the output), cutting all of them also saves the launch for
// those, and wins further out (few: 4 to 40 small items; many: as many as large ones):
//            2 steps      4            8            12           16           24
//   136 few  0.69 / 0.71  0.73 / 0.81  0.77 / 0.88  0.83 / 0.98  0.86 / 1.00  0.92 / 1.04
//   136 many 0.64 / 0.66  0.64 / 0.74  0.66 / 0.79  0.70 / 0.80  0.75 / 0.86  0.80 / 0.87
//   192 few  0.82 / 0.86  0.81 / 0.95  0.86 / 0.98  0.89 / 1.02  0.91 / 1.06  0.94 / 1.11
//   192 many 0.70 / 0.79  0.71 / 0.84  0.74 / 0.90  0.76 / 0.91  0.80 / 0.96  0.84 / 0.99
//   224 few  0.78 / 0.82  0.75 / 0.93  0.81 / 1.08  0.86 / 1.11  0.88 / 1.16  0.92 / 1.24
//   224 many 0.72 / 0.83  0.74 / 0.90  0.79 / 1.02  0.86 / 1.07  0.96 / 1.16  1.02 / 1.21
//   272 few  0.70 / 0.78  0.65 / 0.84  0.67 / 0.92  0.71 / 0.97  0.74 / 0.99  0.78 / 0.99
//   272 many 0.67 / 0.79  0.66 / 0.86  0.67 / 0.86  0.70 / 0.86  0.71 / 0.83  0.71 / 0.84
//   288 few  0.68 / 0.79  0.65 / 0.88  0.68 / 0.94  0.72 / 0.96  0.75 / 0.97  0.79 / 1.01
//   288 many 0.69 / 0.77  0.67 / 0.85  0.68 / 0.91  0.71 / 0.87  0.72 / 0.84  0.73 / 0.84
//   320 few  0.79 / 0.90  0.78 / 0.96  0.80 / 1.01  0.82 / 0.98  0.83 / 1.01  0.84 / 1.05
//   320 many 0.72 / 0.84  0.71 / 0.90  0.77 / 0.90  0.79 / 0.93  0.81 / 0.94  0.83 / 0.97
//   352 few  0.79 / 0.94  0.79 / 1.05  0.78 / 1.04  0.80 / 1.08  0.83 / 1.10  0.84 / 1.14
//   352 many 0.75 / 0.86  0.74 / 0.92  0.74 / 0.97  0.85 / 0.93  0.80 / 1.00  0.85 / 1.00
//   384 few  0.77 / 0.92  0.82 / 1.03  0.82 / 1.12  0.89 / 1.19  0.93 / 1.21  0.97 / 1.26
//   384 many 0.77 / 0.93  0.81 / 1.04  0.84 / 1.04  0.88 / 1.04  0.89 / 1.04  0.89 / 1.07
//   544 few  0.79 / 0.91  0.74 / 1.06  0.80 / 1.13  0.82 / 1.16  0.84 / 1.17  0.88 / 1.21
//   544 many 0.76 / 0.83  0.72 / 0.94  0.80 / 0.96  0.79 / 0.97  0.79 / 0.98  0.94 / 0.98
//   576 few  0.84 / 0.98  0.83 / 1.09  0.91 / 1.18  0.91 / 1.20  0.93 / 1.21  0.96 / 1.27
//   576 many 0.79 / 0.91  0.78 / 1.00  0.88 / 1.02  0.86 / 1.05  0.97 / 1.04  1.01 / 1.05
//   640 few  0.85 / 1.03  0.83 / 1.13  0.92 / 1.23  0.92 / 1.25  0.95 / 1.33  1.25 / 1.37
//   640 many 0.82 / 0.96  0.81 / 1.04  0.88 / 1.10  0.98 / 1.11  1.05 / 1.11  1.12 / 1.07
// Operands are rarely as cold as that in a layer's pass: beside a rim of an eighth to
// a half of the large items its launches gain to the further lines (passes of layers
// and linears whose launches lie between the two, small / large cut: 208 items and 52
// small of 17 steps 1908 / 1960, 224 and 108 of 24 2468 / 2513, 522 and 154 of 20 1992
// / 2034, 528 and 96 of 18 1226 / 1244, 576 and 196 of 18 490 / 508 us).  Beside fewer
// they do not (one product, three sets of operands in turn: 224 and 8 of 20 steps 83 /
// 69, 384 and 8 of 12 104 / 93, 544 and 8 of 24 211 / 187, 576 and 8 of 10 142 / 127,
// 640 and 8 of 5 123 / 110 with an output 1024 wide; square 0.94 to 1.07).
// Lists with items of other lengths among them keep the balanced schedule of
// both classes: rounds say nothing about those (caches as above: 320 items of 3
// and 1 steps 1.12 / 1.06; 16 steps and a few of 8, 269 items 1.04 / 1.15, 286
// items 0.84 / 0.96).
bool cut_small(const cleave_plan* plan, int cus) {
  const int64_t n = static_cast<int64_t>(plan->items[cleave::kTileLarge].size());
  if (n == 0) return false;
  if (2 * n <= cus) return true;
  const int64_t steps = plan->large_steps, over = n % cus;
  const bool equal = steps - plan->large_steps_least <= 1;   // but for a shorter last chunk
  const int64_t rim = static_cast<int64_t>(plan->items[cleave::kTileSmall].size());
  if (!equal || rim > n) return false;
  const bool few = 8 * rim < n, many = 2 * rim > n;
  switch (n / cus) {
    case 0:
      if (rim > 0) return (4 * n <= 3 * cus && steps <= 24) || (8 * n <= 7 * cus && steps <= (few || many ? 12 : 24));
      return 4 * n <= 3 * cus && steps <= 4;
    case 1:
      if (over == 0) return false;
      if (8 * over <= cus) return true;
      if (rim > 0) return (8 * over <= 3 * cus && steps <= 24) || (2 * over <= cus && steps <= (few ? 8 : 12));
      return 4 * over <= cus && steps <= 16;
    case 2:
      if (over == 0) return false;
      if (rim > 0 && few)
        return (8 * over <= cus && steps <= 16) || (4 * over <= cus && steps <= 8) || (2 * over <= cus && steps <= 4);
      if (rim > 0) return (4 * over <= cus && steps <= 24) || (2 * over <= cus && steps <= 8);
      return 8 * over <= cus && steps <= 8;
    default: return false;
  }
}

int execute_impl(cleave_plan* plan, const int64_t* task_ids, int64_t n_ids, const void* A,
                 int64_t lda, int transA, const void* B, int64_t ldb, int transB, int dtype,
                 float* partials, const BatchLayout& bl, void* hip_stream,
                 const AssembleTarget& asm_to = AssembleTarget{}, bool static_scratch = false) {
  if (!plan || !A || !B || (!partials && !asm_to.C)) return CLEAVE_EINVAL;
  if (dtype != CLEAVE_F32 && dtype != CLEAVE_BF16) return CLEAVE_EINVAL;
  if ((transA != 0 && transA != 1) || (transB != 0 && transB != 1)) return CLEAVE_EINVAL;
  if ((task_ids == nullptr) != (n_ids == 0) || n_ids < 0) return CLEAVE_EINVAL;
  if (lda < (transA ? plan->M : plan->K) || ldb < (transB ? plan->K : plan->N)) return CLEAVE_EINVAL;
  const int eb = dtype == CLEAVE_BF16 ? 2 : 4;
  if (!aligned(A, eb) || !aligned(B, eb) || !aligned(partials, 4)) return CLEAVE_EINVAL;   // null partials: assemble mode
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);

  int cus = 0;
  int rc = compute_units(&cus);
  if (rc != CLEAVE_OK) return rc;
  int dev = 0;
  CLEAVE_HIP(hipGetDevice(&dev));
  if (static_scratch) {
    // this entry point never allocates: the tables must be on the device already
    if (plan->device != dev) return CLEAVE_EINVAL;
  } else {
    rc = ensure_uploaded(plan);
    if (rc != CLEAVE_OK) return rc;
  }

  // The direct kernel: bf16, every 16 bytes that it fetches (8 elements along the
  // operand's rows as stored) belong to one chunk and one tile and lie on a
  // 16-byte boundary; rows of the output in whole eights.  An operand stored
  // with the inner dimension across its rows takes any chunk, the other kind any
  // tile row.  Chunks that end within a K step against the general kernel (us):
  // 4096 x 4096 x 4128 in 4 splits 230 / 175, 4096 x 8192 x 1032 101 / 71, 8192 x
  // 3072 x 800 in 4 126 / 98, 512 x 512 x 200 5.2 / 4.4; odd chunks of two operands
  // with the inner dimension across, 3000 x 2504 x 3001 in 4 77 / 54; odd rows, 3001
  // x 2504 x 1024 in 4 37 / 30.
  const int e = 16 / eb;
  const bool direct = dtype == CLEAVE_BF16 && plan->all_n_mult8 && (transA ? plan->all_m_mult8 : plan->all_k_mult8) &&
                      (!transB || plan->all_k_mult8) &&
                      lda % e == 0 && ldb % e == 0 && aligned(A, 16) && aligned(B, 16) &&
                      // in-tile byte offsets are kept in 32 bits
                      lda * eb < (int64_t{1} << 22) && ldb * eb < (int64_t{1} << 22) &&
                      offsets_multiple_of(bl.a, bl.shape, e) && offsets_multiple_of(bl.b, bl.shape, e);
  // An operand of the general kernel's 16-byte loads needs that much between the start of a
  // stored row and the end of any chunk (K-contiguous) or row (otherwise), and
  // in-tile byte offsets (up to 128 rows) that fit 32 bits.
  const bool a_elements = (transA ? plan->M : plan->min_k_end) < e || lda * eb >= (int64_t{1} << 25);
  const bool b_elements = (transB ? plan->min_k_end : plan->N) < e || ldb * eb >= (int64_t{1} << 25);

  const cleave::WorkItem* d_lists[cleave::kNumTileClasses] = {plan->d_items[0], plan->d_items[1]};
  int64_t counts[cleave::kNumTileClasses] = {static_cast<int64_t>(plan->items[0].size()),
                                             static_cast<int64_t>(plan->items[1].size())};
  int64_t steps[cleave::kNumTileClasses] = {plan->items_steps[0], plan->items_steps[1]};   // whole K steps of a list's items
  cleave::ListShape shapes[cleave::kNumTileClasses] = {plan->shape, plan->shape};   // (the general kernel runs all tasks, or a subset)
  // which of the plan's lists a class runs from (-1: a subset's own list)
  int list_of[cleave::kNumTileClasses] = {task_ids ? -1 : 0, task_ids ? -1 : 1};
  if (!task_ids && (!direct || cut_small(plan, cus))) {
    list_of[cleave::kTileSmall] = cleave::kNumTileClasses;
    d_lists[cleave::kTileLarge] = nullptr;
    counts[cleave::kTileLarge] = 0;
    d_lists[cleave::kTileSmall] = plan->d_items_fine;
    counts[cleave::kTileSmall] = static_cast<int64_t>(plan->items_fine.size());
    steps[cleave::kTileSmall] = plan->items_steps[cleave::kNumTileClasses];
  }
  // Subset launches: the work-item lists are written on the device, from the
  // task records, into a slice of memory the plan set aside when its tables
  // were uploaded -- stream-ordered, no host wait, no copy, no allocation.
  std::unique_lock<std::mutex> subset_lock;
  int64_t slice_begin = -1, slice_total = 0;
  if (task_ids) {
    subset_lock = std::unique_lock<std::mutex>(plan->subset.mu);
    SubsetLayout layout;
    rc = layout_subset(plan, task_ids, n_ids, cus, &layout);
    if (rc != CLEAVE_OK) return rc;
    slice_total = layout.total();
    cleave::WorkItem* slice = nullptr;
    if (static_scratch) {
      // the device's fixed array, from its start: whatever an earlier call left there is overwritten
      if (slice_total > kStaticScratchItems) return CLEAVE_ELIMIT;
      slice = g_static_scratch[dev];
    } else {
      hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
      CLEAVE_HIP(hipStreamIsCapturing(stream, &capture));
      rc = acquire_subset_slice(plan->subset, slice_total, capture != hipStreamCaptureStatusNone, &slice,
                                &slice_begin);
      if (rc != CLEAVE_OK) return rc;
    }
    rc = expand_subset(plan, task_ids, n_ids, layout, slice, stream);
    if (rc != CLEAVE_OK) {
      if (!static_scratch) (void)release_subset_slice(plan->subset, slice_begin, slice_total, stream);
      return rc;
    }
    int64_t pos = 0;
    for (int c = 0; c < cleave::kNumTileClasses; ++c) {
      d_lists[c] = slice + pos;
      steps[c] = layout.steps[c];
      shapes[c] = layout.shapes[c];
      counts[c] = layout.counts[c];
      pos += counts[c];
    }
  }

  // whatever has been enqueued reads the slice: mark it even if a later launch fails
  const auto launch_failed = [&](hipError_t e) {
    if (task_ids && !static_scratch) (void)release_subset_slice(plan->subset, slice_begin, slice_total, stream);
    return hip_fail(e);
  };
  int64_t most = -1;
  for (int c = 0; c < cleave::kNumTileClasses; ++c) {
    if (counts[c] == 0) continue;
    cleave::ExecuteArgs args{};
    args.items = d_lists[c];
    args.n_items = counts[c];
    args.A = A;
    args.B = B;
    args.lda = lda;
    args.ldb = ldb;
    args.transA = transA;
    args.transB = transB;
    args.partials = partials;
    args.batch = bl.shape;
    args.a_at = bl.a;
    args.b_at = bl.b;
    args.c_at = bl.c;
    args.C = asm_to.C;
    args.M = plan->M;
    args.N = plan->N;
    args.K = plan->K;
    args.ldc = asm_to.ldc;
    args.stream_below_k = task_ids ? 0 : streamed_below(plan, asm_to);
    args.c_bf16 = asm_to.out_dtype == CLEAVE_BF16 ? 1 : 0;
    const bool large = c == cleave::kTileLarge;
    if (direct) {
      // Persistent workgroups, as many as the chip holds at once: each walks
      // the item list with the grid as stride and fetches the head of its next
      // item while it stores the current one.
      const cleave::DirectShape shape = direct_shape(c, counts[c], cus);
      const int64_t resident = static_cast<int64_t>(cus) * cleave::direct_workgroups_per_cu(shape);
      const int grid = static_cast<int>(std::min<int64_t>(counts[c], resident));
      // items of unequal length: the schedule made for this grid when the tables were uploaded
      const int list = list_of[c];
      args.wg_ranges = (list >= 0 && plan->wg_ranges_grid[list] == grid)
                           ? plan->d_wg_ranges[list] : nullptr;
      if (args.wg_ranges && list == cleave::kNumTileClasses) args.items += counts[c];   // behind the list as laid out
      const hipError_t he = cleave::launch_execute_direct(args, shape, plan->chunk_tails, grid, stream);
      if (he != hipSuccess) return launch_failed(he);
      if (counts[c] > most) plan->last_kernel = direct_kernel_name(shape, transA, transB);
    } else {
      // in-tile byte offsets (256 rows) stay within 32 bits
      const bool by_k = !transA && transB && !a_elements && !b_elements && lda * eb < (int64_t{1} << 24) &&
                        ldb * eb < (int64_t{1} << 24);
      const int64_t items = counts[c] * (large ? 4 : 1);
      cleave::GeneralLoads how{
          general_tile(dtype, !transA && transB, items, shapes[c], large && dtype == CLEAVE_BF16 && by_k ? counts[c] : 0,
                       steps[c], cus),
          a_elements, b_elements, shapes[c], cus};
      if (how.tile == cleave::kTileWide && cleave::four_waves(dtype, transA, transB, items, shapes[c], cus))
        how.tile = cleave::kTileWide4;
      if (how.tile == cleave::kTileNarrow && cleave::runs_lone(dtype, c, counts[c], shapes[c], cus))
        how.tile = cleave::kTileLone;
      const hipError_t he = cleave::launch_execute(args, dtype, c, how, stream);
      if (he != hipSuccess) return launch_failed(he);
      if (counts[c] > most) plan->last_kernel = kernel_name(dtype, how, transA, transB);
    }
    most = std::max(most, counts[c]);
  }
  if (task_ids && !static_scratch) return release_subset_slice(plan->subset, slice_begin, slice_total, stream);
  return CLEAVE_OK;
}

}  // namespace

extern "C" int cleave_execute(cleave_plan* plan, const int64_t* task_ids, int64_t n_ids,
                              const void* A, int64_t lda, int transA, const void* B, int64_t ldb,
                              int transB, int dtype, float* partials, void* hip_stream) {
  if (plan && plan->batch > 0) return CLEAVE_EINVAL;   // batched plans use the batched call
  return execute_impl(plan, task_ids, n_ids, A, lda, transA, B, ldb, transB, dtype, partials,
                      BatchLayout{}, hip_stream);
}

extern "C" int cleave_execute_noalloc(cleave_plan* plan, const int64_t* task_ids, int64_t n_ids,
                                      const void* A, int64_t lda, int transA, const void* B,
                                      int64_t ldb, int transB, int dtype, float* partials,
                                      void* hip_stream) {
  if (plan && plan->batch > 0) return CLEAVE_EINVAL;
  return execute_impl(plan, task_ids, n_ids, A, lda, transA, B, ldb, transB, dtype, partials,
                      BatchLayout{}, hip_stream, AssembleTarget{}, true);
}

extern "C" int cleave_execute_batched(cleave_plan* plan, const int64_t* task_ids, int64_t n_ids,
                                      const void* A, int64_t lda, int transA, int64_t a_outer,
                                      int64_t a_inner, const void* B, int64_t ldb, int transB,
                                      int64_t b_outer, int64_t b_inner, int64_t n_inner, int dtype,
                                      float* partials, void* hip_stream) {
  if (!plan || plan->batch < 1) return CLEAVE_EINVAL;
  if (n_inner < 1 || n_inner > std::numeric_limits<uint32_t>::max() || plan->batch % n_inner != 0)
    return CLEAVE_EINVAL;
  if (a_outer < 0 || a_inner < 0 || b_outer < 0 || b_inner < 0) return CLEAVE_EINVAL;
  return execute_impl(plan, task_ids, n_ids, A, lda, transA, B, ldb, transB, dtype, partials,
                      strided_layout(n_inner, a_outer, a_inner, b_outer, b_inner, 0, 0), hip_stream);
}

extern "C" int cleave_execute_grouped(cleave_plan* plan, const int64_t* task_ids, int64_t n_ids,
                                      int64_t n_members, const void* const* A_list, int64_t lda,
                                      int transA,
                                      const void* const* B_list, int64_t ldb, int transB, int dtype,
                                      float* partials, void* hip_stream) {
  if (!plan || plan->batch < 1 || plan->batch > cleave::kMaxGroup || n_members != plan->batch)
    return CLEAVE_EINVAL;
  if (dtype != CLEAVE_F32 && dtype != CLEAVE_BF16) return CLEAVE_EINVAL;
  const int eb = dtype == CLEAVE_BF16 ? 2 : 4;
  BatchLayout bl;
  bl.shape.n_group = static_cast<uint32_t>(plan->batch);
  const void* A = nullptr;
  const void* B = nullptr;
  int rc = group_offsets(A_list, plan->batch, eb, &bl.a, &A);
  if (rc != CLEAVE_OK) return rc;
  rc = group_offsets(B_list, plan->batch, eb, &bl.b, &B);
  if (rc != CLEAVE_OK) return rc;
  return execute_impl(plan, task_ids, n_ids, A, lda, transA, B, ldb, transB, dtype, partials, bl,
                      hip_stream);
}

extern "C" int cleave_execute_assemble(cleave_plan* plan, const int64_t* task_ids, int64_t n_ids,
                                       const void* A, int64_t lda, int transA, int64_t a_outer,
                                       int64_t a_inner, const void* B, int64_t ldb, int transB,
                                       int64_t b_outer, int64_t b_inner, int64_t n_inner, int dtype,
                                       void* C, int64_t ldc, int64_t c_outer, int64_t c_inner,
                                       int out_dtype, void* hip_stream) {
  if (!plan || !C) return CLEAVE_EINVAL;
  if (out_dtype != CLEAVE_F32 && out_dtype != CLEAVE_BF16) return CLEAVE_EINVAL;
  if (ldc < plan->N || !aligned(C, out_dtype == CLEAVE_BF16 ? 2 : 4)) return CLEAVE_EINVAL;
  // a block is the finished output only if its task covers the whole inner dimension
  for (const cleave_task& t : plan->tasks)
    if (t.ksplit_cnt != 1) return CLEAVE_EINVAL;
  BatchLayout bl;
  if (plan->batch > 0) {
    if (n_inner < 1 || n_inner > std::numeric_limits<uint32_t>::max() || plan->batch % n_inner != 0)
      return CLEAVE_EINVAL;
    if (a_outer < 0 || a_inner < 0 || b_outer < 0 || b_inner < 0 || c_outer < 0 || c_inner < 0)
      return CLEAVE_EINVAL;
    bl = strided_layout(n_inner, a_outer, a_inner, b_outer, b_inner, c_outer, c_inner);
  } else if (n_inner != 0 || a_outer || a_inner || b_outer || b_inner || c_outer || c_inner) {
    return CLEAVE_EINVAL;   // strides belong to batched plans
  }
  AssembleTarget to;
  to.C = C;
  to.ldc = ldc;
  to.out_dtype = out_dtype;
  return execute_impl(plan, task_ids, n_ids, A, lda, transA, B, ldb, transB, dtype, nullptr, bl,
                      hip_stream, to);
}

namespace {

// Which operator consumes the aggregated values.
struct ReduceEpilogue {
  const void* residual = nullptr;          // C = sum + residual
  const cleave::AdamArgs* adam = nullptr;  // Adam update of adam->w (C unused)
  const cleave::AdamGroupOffsets* adam_group = nullptr;   // with adam: one set of arrays per member
};

int reduce_impl(cleave_plan* plan, const float* partials, void* C, int64_t ldc, int out_dtype,
                const BatchLayout& bl, void* hip_stream,
                const ReduceEpilogue& epi = ReduceEpilogue{}, bool members_aligned = true) {
  if (!plan || !partials || !C) return CLEAVE_EINVAL;
  if (out_dtype != CLEAVE_F32 && out_dtype != CLEAVE_BF16) return CLEAVE_EINVAL;
  if (ldc < plan->N) return CLEAVE_EINVAL;
  const int ob = out_dtype == CLEAVE_BF16 ? 2 : 4;
  if (!aligned(partials, 4) || !aligned(C, ob)) return CLEAVE_EINVAL;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);

  int rc = ensure_uploaded(plan);
  if (rc != CLEAVE_OK) return rc;

  bool vec = plan->all_n_mult4 && ldc % 4 == 0 && aligned(partials, 16) && aligned(C, 4 * ob) &&
             offsets_multiple_of(bl.c, bl.shape, 4) && members_aligned;
  if (epi.residual) vec = vec && aligned(epi.residual, 4 * ob);
  if (epi.adam)
    vec = vec && aligned(epi.adam->m, 16) && aligned(epi.adam->v, 16) &&
          (!epi.adam->w_bf16 || aligned(epi.adam->w_bf16, 8));
  cleave::ReduceArgs args{};
  args.items = plan->d_reduce_items;
  args.n_items = plan->reduce_runs;
  args.partials = partials;
  args.C = C;
  args.ldc = ldc;
  args.batch = bl.shape;
  args.c_at = bl.c;
  // one workgroup per reduce item (the kernel loops only if the grid is capped)
  const int grid = static_cast<int>(std::min<int64_t>(args.n_items, int64_t{1} << 20));
  if (epi.adam && epi.adam_group) {
    CLEAVE_HIP(cleave::launch_reduce_adam_grouped(args, *epi.adam, *epi.adam_group, vec, grid, stream));
  } else if (epi.adam) {
    CLEAVE_HIP(cleave::launch_reduce_adam(args, *epi.adam, vec, grid, stream));
  } else if (epi.residual) {
    CLEAVE_HIP(cleave::launch_reduce_residual(args, epi.residual, out_dtype, vec, grid, stream));
  } else {
    CLEAVE_HIP(cleave::launch_reduce(args, out_dtype, vec, grid, stream));
  }
  return CLEAVE_OK;
}

}  // namespace

extern "C" int cleave_reduce_residual(cleave_plan* plan, const float* partials, const void* R,
                                      void* C, int64_t ldc, int out_dtype, void* hip_stream) {
  if (!R || (plan && plan->batch > 0)) return CLEAVE_EINVAL;
  if (out_dtype != CLEAVE_F32 && out_dtype != CLEAVE_BF16) return CLEAVE_EINVAL;
  if (!aligned(R, out_dtype == CLEAVE_BF16 ? 2 : 4)) return CLEAVE_EINVAL;
  ReduceEpilogue epi;
  epi.residual = R;
  return reduce_impl(plan, partials, C, ldc, out_dtype, BatchLayout{}, hip_stream, epi);
}

extern "C" int cleave_reduce_adam(cleave_plan* plan, const float* partials, float* w, float* m,
                                  float* v, void* w_bf16, int64_t ld, float lr, float beta1,
                                  float beta2, float eps, float weight_decay, int64_t step,
                                  void* hip_stream) {
  if (!w || !m || !v || (plan && plan->batch > 0)) return CLEAVE_EINVAL;
  if (step < 1 || !(beta1 >= 0.0f && beta1 < 1.0f) || !(beta2 >= 0.0f && beta2 < 1.0f) ||
      !(eps >= 0.0f) || !(lr == lr) || !(weight_decay == weight_decay))
    return CLEAVE_EINVAL;
  if (!aligned(m, 4) || !aligned(v, 4) || !aligned(w_bf16, 2)) return CLEAVE_EINVAL;
  cleave::AdamArgs h{};
  h.w = w;
  h.m = m;
  h.v = v;
  h.w_bf16 = static_cast<uint16_t*>(w_bf16);
  h.lr = lr;
  h.beta1 = beta1;
  h.beta2 = beta2;
  h.eps = eps;
  h.weight_decay = weight_decay;
  h.inv_bias1 = static_cast<float>(1.0 / (1.0 - std::pow(static_cast<double>(beta1), static_cast<double>(step))));
  h.inv_bias2 = static_cast<float>(1.0 / (1.0 - std::pow(static_cast<double>(beta2), static_cast<double>(step))));
  ReduceEpilogue epi;
  epi.adam = &h;
  // the fp32 master weight takes C's place in the common checks (pointer, leading dimension)
  return reduce_impl(plan, partials, w, ld, CLEAVE_F32, BatchLayout{}, hip_stream, epi);
}

extern "C" int cleave_reduce_adam_grouped(cleave_plan* plan, const float* partials, int64_t n_members,
                                          float* const* w_list, float* const* m_list,
                                          float* const* v_list, void* const* w_bf16_list, int64_t ld,
                                          float lr, float beta1, float beta2, float eps,
                                          float weight_decay, int64_t step, void* hip_stream) {
  if (!plan || plan->batch < 1 || plan->batch > cleave::kMaxGroup || n_members != plan->batch)
    return CLEAVE_EINVAL;
  if (!w_list || !m_list || !v_list) return CLEAVE_EINVAL;
  if (step < 1 || !(beta1 >= 0.0f && beta1 < 1.0f) || !(beta2 >= 0.0f && beta2 < 1.0f) ||
      !(eps >= 0.0f) || !(lr == lr) || !(weight_decay == weight_decay))
    return CLEAVE_EINVAL;
  cleave::AdamGroupOffsets at{};
  bool all16 = true;
  for (int64_t g = 0; g < n_members; ++g) {
    if (!w_list[g] || !m_list[g] || !v_list[g] || (w_bf16_list && !w_bf16_list[g])) return CLEAVE_EINVAL;
    if (!aligned(w_list[g], 4) || !aligned(m_list[g], 4) || !aligned(v_list[g], 4) ||
        (w_bf16_list && !aligned(w_bf16_list[g], 2)))
      return CLEAVE_EINVAL;
    all16 = all16 && aligned(w_list[g], 16) && aligned(m_list[g], 16) && aligned(v_list[g], 16) &&
            (!w_bf16_list || aligned(w_bf16_list[g], 8));
    at.w[g] = w_list[g] - w_list[0];
    at.m[g] = m_list[g] - m_list[0];
    at.v[g] = v_list[g] - v_list[0];
    at.w_bf16[g] = w_bf16_list ? static_cast<uint16_t*>(w_bf16_list[g]) - static_cast<uint16_t*>(w_bf16_list[0]) : 0;
  }
  cleave::AdamArgs h{};
  h.w = w_list[0];
  h.m = m_list[0];
  h.v = v_list[0];
  h.w_bf16 = w_bf16_list ? static_cast<uint16_t*>(w_bf16_list[0]) : nullptr;
  h.lr = lr;
  h.beta1 = beta1;
  h.beta2 = beta2;
  h.eps = eps;
  h.weight_decay = weight_decay;
  h.inv_bias1 = static_cast<float>(1.0 / (1.0 - std::pow(static_cast<double>(beta1), static_cast<double>(step))));
  h.inv_bias2 = static_cast<float>(1.0 / (1.0 - std::pow(static_cast<double>(beta2), static_cast<double>(step))));
  ReduceEpilogue epi;
  epi.adam = &h;
  epi.adam_group = &at;
  BatchLayout bl;
  bl.shape.n_group = static_cast<uint32_t>(plan->batch);   // c_at stays zero: every array has its own table
  // reduce_impl's vector-path test looks at h's (member 0's) arrays; the members must agree
  // (a member whose arrays are not 16-byte aligned sends the whole launch down the element path)
  return reduce_impl(plan, partials, h.w, ld, CLEAVE_F32, bl, hip_stream, epi, all16);
}

extern "C" int cleave_reduce(cleave_plan* plan, const float* partials, void* C, int64_t ldc,
                             int out_dtype, void* hip_stream) {
  if (plan && plan->batch > 0) return CLEAVE_EINVAL;
  return reduce_impl(plan, partials, C, ldc, out_dtype, BatchLayout{}, hip_stream);
}

extern "C" int cleave_reduce_batched(cleave_plan* plan, const float* partials, void* C, int64_t ldc,
                                     int64_t c_outer, int64_t c_inner, int64_t n_inner,
                                     int out_dtype, void* hip_stream) {
  if (!plan || plan->batch < 1) return CLEAVE_EINVAL;
  if (n_inner < 1 || n_inner > std::numeric_limits<uint32_t>::max() || plan->batch % n_inner != 0)
    return CLEAVE_EINVAL;
  if (c_outer < 0 || c_inner < 0) return CLEAVE_EINVAL;
  return reduce_impl(plan, partials, C, ldc, out_dtype,
                     strided_layout(n_inner, 0, 0, 0, 0, c_outer, c_inner), hip_stream);
}

extern "C" int cleave_reduce_grouped(cleave_plan* plan, const float* partials, int64_t n_members,
                                     void* const* C_list, int64_t ldc, int out_dtype,
                                     void* hip_stream) {
  if (!plan || plan->batch < 1 || plan->batch > cleave::kMaxGroup || n_members != plan->batch)
    return CLEAVE_EINVAL;
  if (out_dtype != CLEAVE_F32 && out_dtype != CLEAVE_BF16) return CLEAVE_EINVAL;
  BatchLayout bl;
  bl.shape.n_group = static_cast<uint32_t>(plan->batch);
  const void* C = nullptr;
  const int rc = group_offsets(C_list, plan->batch, out_dtype == CLEAVE_BF16 ? 2 : 4, &bl.c, &C);
  if (rc != CLEAVE_OK) return rc;
  return reduce_impl(plan, partials, const_cast<void*>(C), ldc, out_dtype, bl, hip_stream);
}

#ifndef CLEAVE_AGG_ELEMS
#define CLEAVE_AGG_ELEMS 8192
#endif

namespace {

// Host tables of the returned-block check (built once per plan) and their
// device copies plus scratch (once per device the plan is used on).
int ensure_verify_tables_host(cleave_plan* p) {
  using cleave::Segment;
  if (!p->verify) {
    cleave::VerifyTables* v = new (std::nothrow) cleave::VerifyTables;
    if (!v) return CLEAVE_ENOMEM;
    try {
      std::map<std::pair<uint32_t, uint32_t>, uint32_t> rows, cols;
      // Elements of a partial block per bilinear item: runs long enough to stream, as
      // short as the last round of workgroups needs.  us, runs of 8 K / 16 K / 32 K: 17 M
      // elements in all 23.4 / 20.1 / 21.8, 67 M 71.8 / 64.4 / 67.4, behind the launch that
      // wrote them 189.4 / 187.9 / 191.4, 134 M 113 / 101 / 104, 180 M 174 / 139 / 144, 268 M
      // 208 / 185 / 188; 451 M in 8 splits of 4 MiB blocks 421 / 336 / 330.
      const uint32_t kElemsPerItem = p->partial_elems >= (int64_t{384} << 20) ? 32768u : 16384u;
      v->task_first_item.push_back(0);
      for (const cleave_task& t : p->tasks) {
        auto ri = rows.emplace(std::make_pair(t.m0, t.m_len), static_cast<uint32_t>(rows.size()));
        if (ri.second) v->row_segs.push_back(Segment{t.m0, t.m_len});
        v->task_row_seg.push_back(ri.first->second);
        auto ci = cols.emplace(std::make_pair(t.n0, t.n_len), static_cast<uint32_t>(cols.size()));
        if (ci.second) v->col_segs.push_back(Segment{t.n0, t.n_len});
        v->task_col_seg.push_back(ci.first->second);
        const uint32_t rows_per = std::max<uint32_t>(1, kElemsPerItem / t.n_len);
        for (uint32_t r0 = 0; r0 < t.m_len; r0 += rows_per)
          v->items.push_back(cleave::make_verify_item(t, r0, std::min(rows_per, t.m_len - r0)));
        v->max_ksplit = std::max(v->max_ksplit, t.ksplit_cnt);
        if (v->items.size() > std::numeric_limits<uint32_t>::max()) {
          delete v;
          return CLEAVE_EINVAL;
        }
        v->task_first_item.push_back(static_cast<uint32_t>(v->items.size()));
      }
      for (const std::vector<Segment>* segs : {&v->row_segs, &v->col_segs})
        for (const Segment& sg : *segs) {
          v->segs_mult8 &= ((sg.start | sg.len) % 8 == 0);
          v->segs_mult4 &= ((sg.start | sg.len) % 4 == 0);
        }
    } catch (const std::bad_alloc&) {
      delete v;
      return CLEAVE_ENOMEM;
    }
    p->verify = v;
  }
  return CLEAVE_OK;
}

int ensure_verify_tables(cleave_plan* p) {
  int rc = ensure_verify_tables_host(p);
  if (rc != CLEAVE_OK) return rc;
  cleave::VerifyTables* v = p->verify;
  if (v->d_items || p->tasks.empty()) return CLEAVE_OK;
  rc = upload_vector(v->row_segs, &v->d_row_segs);
  if (rc == CLEAVE_OK) rc = upload_vector(v->col_segs, &v->d_col_segs);
  if (rc == CLEAVE_OK) rc = upload_vector(v->task_row_seg, &v->d_task_row_seg);
  if (rc == CLEAVE_OK) rc = upload_vector(v->task_col_seg, &v->d_task_col_seg);
  if (rc == CLEAVE_OK) rc = upload_vector(v->task_first_item, &v->d_task_first_item);
  if (rc == CLEAVE_OK) rc = upload_vector(v->items, &v->d_items);
  if (rc == CLEAVE_OK) {
    const size_t members = p->batch > 0 ? static_cast<size_t>(p->batch) : 1;
    const size_t proj = 2 * (v->row_segs.size() + v->col_segs.size()) * static_cast<size_t>(p->K) * members;
    hipError_t e = hipMalloc(reinterpret_cast<void**>(&v->d_proj), proj * sizeof(double));
    if (e == hipSuccess)
      e = hipMalloc(reinterpret_cast<void**>(&v->d_item_sums), v->items.size() * sizeof(double));
    if (e == hipErrorOutOfMemory) rc = CLEAVE_ENOMEM;
    else if (e != hipSuccess) rc = hip_fail(e);
  }
  if (rc != CLEAVE_OK) free_verify_device(v);
  return rc;
}

// Tables of the fused check + aggregation (first fused call on the plan, after
// ensure_verify_tables): runs of rows of ~kAggElemsPerItem output elements.
int ensure_aggregate_tables(cleave_plan* p) {
  cleave::VerifyTables* v = p->verify;
  if (v->d_agg_items || p->tasks.empty()) return CLEAVE_OK;
  if (v->agg_first_item.empty()) {
    try {
      constexpr uint32_t kAggElemsPerItem = CLEAVE_AGG_ELEMS;
      uint64_t slots = 0;
      v->agg_first_item.push_back(0);
      for (const cleave_task& t : p->tasks) {
        const uint32_t rows_per = std::max<uint32_t>(1, kAggElemsPerItem / t.n_len);
        const uint32_t runs = (t.m_len + rows_per - 1) / rows_per;
        for (uint32_t j = 0; t.ksplit_idx == 0 && j < runs; ++j) {
          const uint32_t r0 = j * rows_per;
          cleave::VerifyItem item = cleave::make_verify_item(t, r0, std::min(rows_per, t.m_len - r0));
          item.slot = static_cast<uint32_t>(slots) + j;
          item.slot_step = runs;
          v->agg_items.push_back(item);
        }
        slots += runs;
        if (slots > std::numeric_limits<uint32_t>::max()) {
          v->agg_items.clear();
          v->agg_first_item.clear();
          return CLEAVE_EINVAL;
        }
        v->agg_first_item.push_back(static_cast<uint32_t>(slots));
      }
    } catch (const std::bad_alloc&) {
      v->agg_items.clear();
      v->agg_first_item.clear();
      return CLEAVE_ENOMEM;
    }
  }
  int rc = upload_vector(v->agg_items, &v->d_agg_items);
  if (rc == CLEAVE_OK) rc = upload_vector(v->agg_first_item, &v->d_agg_first_item);
  if (rc == CLEAVE_OK) {
    const hipError_t e = hipMalloc(reinterpret_cast<void**>(&v->d_agg_item_sums),
                                   static_cast<size_t>(v->agg_first_item.back()) * sizeof(double));
    if (e == hipErrorOutOfMemory) rc = CLEAVE_ENOMEM;
    else if (e != hipSuccess) rc = hip_fail(e);
  }
  if (rc != CLEAVE_OK) {
    for (void* q : {static_cast<void*>(v->d_agg_items), static_cast<void*>(v->d_agg_first_item),
                    static_cast<void*>(v->d_agg_item_sums)})
      if (q) (void)hipFree(q);
    v->d_agg_items = nullptr;
    v->d_agg_first_item = nullptr;
    v->d_agg_item_sums = nullptr;
  }
  return rc;
}

}  // namespace

namespace {

// Where the fused pass writes the aggregated output (C == nullptr: check only).
struct AggregateTarget {
  void* C = nullptr;
  int64_t ldc = 0;
  int out_dtype = CLEAVE_F32;
};

int verify_impl(cleave_plan* plan, const void* A, int64_t lda, int transA, const void* B, int64_t ldb,
                int transB, int dtype, const float* partials, const float* r, const float* s, double tol,
                double* lhs, double* rhs, double* scale, int32_t* accept, const BatchLayout& bl,
                void* hip_stream, const AggregateTarget& agg = AggregateTarget{}) {
  if (!plan || !A || !B || !partials || !r || !s || !accept) return CLEAVE_EINVAL;
  if (dtype != CLEAVE_F32 && dtype != CLEAVE_BF16) return CLEAVE_EINVAL;
  if ((transA != 0 && transA != 1) || (transB != 0 && transB != 1)) return CLEAVE_EINVAL;
  if (lda < (transA ? plan->M : plan->K) || ldb < (transB ? plan->K : plan->N)) return CLEAVE_EINVAL;
  if (!(tol >= 0.0)) return CLEAVE_EINVAL;   // also refuses NaN
  const int eb = dtype == CLEAVE_BF16 ? 2 : 4;
  if (!aligned(A, eb) || !aligned(B, eb) || !aligned(partials, 4) || !aligned(r, 4) ||
      !aligned(s, 4) || !aligned(accept, 4) || !aligned(lhs, 8) || !aligned(rhs, 8) ||
      !aligned(scale, 8))
    return CLEAVE_EINVAL;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);

  int rc = ensure_uploaded(plan);
  if (rc != CLEAVE_OK) return rc;
  rc = ensure_verify_tables(plan);
  if (rc != CLEAVE_OK) return rc;
  cleave::VerifyTables* v = plan->verify;
  if (plan->tasks.empty()) return CLEAVE_OK;

  const int64_t K = plan->K;
  const bool batched = plan->batch > 0;
  const int n_members = batched ? static_cast<int>(plan->batch) : 1;
  const int e = 16 / eb;   // elements per 16-byte load
  const bool segs_ok = e == 8 ? v->segs_mult8 : v->segs_mult4;
  const size_t row_proj = v->row_segs.size() * static_cast<size_t>(K) * static_cast<size_t>(n_members);
  const size_t col_proj = v->col_segs.size() * static_cast<size_t>(K) * static_cast<size_t>(n_members);
  double* U = v->d_proj;
  double* U_abs = U + row_proj;
  double* V = U_abs + row_proj;
  double* V_abs = V + col_proj;

  // op(A)[i][k]: stored M x K (transA = 0) -> the summed row index strides;
  // stored K x M (transA = 1) -> it is contiguous.  op(B)[k][j]: stored K x N
  // (transB = 0) -> the summed column index is contiguous; stored N x K -> it
  // strides.
  const bool a_contig = transA != 0;
  const bool b_contig = transB == 0;
  // members' probe vectors follow each other: r is n_members x M, s is n_members x N
  const int64_t r_stride = batched ? plan->M : 0, s_stride = batched ? plan->N : 0;
  const bool a_vec = aligned(A, 16) && lda % e == 0 && offsets_multiple_of(bl.a, bl.shape, e) &&
                     (a_contig ? (segs_ok && aligned(r, 16) && r_stride % 4 == 0) : K % e == 0);
  const bool b_vec = aligned(B, 16) && ldb % e == 0 && offsets_multiple_of(bl.b, bl.shape, e) &&
                     (b_contig ? (segs_ok && aligned(s, 16) && s_stride % 4 == 0) : K % e == 0);
  const bool p_vec = plan->all_n_mult4 && aligned(partials, 16) && aligned(s, 16) && s_stride % 4 == 0;
  cleave::VerifyPassArgs pass{};
  pass.A = cleave::ProjectArgs{A, lda, v->d_row_segs, static_cast<int>(v->row_segs.size()), r, U, U_abs, K,
                               n_members, r_stride, bl.shape, bl.a};
  pass.B = cleave::ProjectArgs{B, ldb, v->d_col_segs, static_cast<int>(v->col_segs.size()), s, V, V_abs, K,
                               n_members, s_stride, bl.shape, bl.b};
  pass.bil = cleave::BilinearArgs{v->d_items, static_cast<int64_t>(v->items.size()),
                                  partials, r, s, v->d_item_sums, batched ? 1 : 0, r_stride, s_stride};
  const uint32_t* first_item = v->d_task_first_item;
  const double* item_sums = v->d_item_sums;
  if (agg.C) {
    rc = ensure_aggregate_tables(plan);
    if (rc != CLEAVE_OK) return rc;
    first_item = v->d_agg_first_item;
    item_sums = v->d_agg_item_sums;
    const int ob = agg.out_dtype == CLEAVE_BF16 ? 2 : 4;
    const bool c_vec = agg.ldc % 4 == 0 && aligned(agg.C, 4 * ob);
    cleave::VerifyReducePassArgs fused{};
    fused.A = pass.A;
    fused.B = pass.B;
    fused.bil = pass.bil;
    fused.bil.item_sums = v->d_agg_item_sums;
    fused.agg = cleave::AggregateArgs{v->d_agg_items, static_cast<int64_t>(v->agg_items.size()), agg.C, agg.ldc, agg.out_dtype == CLEAVE_BF16 ? 1 : 0,
                                      agg.out_dtype == CLEAVE_F32 && cleave::streamed_sum(plan->M * plan->N, plan->partial_elems)};
    CLEAVE_HIP(cleave::launch_verify_reduce_pass(fused, dtype, a_contig, b_contig,
                                                 a_vec && b_vec && p_vec && c_vec, stream));
  } else {
    CLEAVE_HIP(cleave::launch_verify_pass(pass, dtype, a_contig, b_contig, a_vec && b_vec && p_vec, stream));
  }

  cleave::VerdictArgs va{plan->d_tasks, static_cast<int64_t>(plan->tasks.size()),
                         v->d_task_row_seg, v->d_task_col_seg, first_item,
                         item_sums, U, U_abs, V, V_abs, K, batched ? 1 : 0,
                         static_cast<int>(v->row_segs.size()), static_cast<int>(v->col_segs.size()),
                         tol, lhs, rhs, scale, accept};
  CLEAVE_HIP(cleave::launch_verdict(va, stream));
  return CLEAVE_OK;
}

}  // namespace

extern "C" int cleave_verify(cleave_plan* plan, const void* A, int64_t lda, int transA,
                             const void* B, int64_t ldb, int transB, int dtype,
                             const float* partials, const float* r, const float* s, double tol,
                             double* lhs, double* rhs, double* scale, int32_t* accept,
                             void* hip_stream) {
  if (plan && plan->batch > 0) return CLEAVE_EINVAL;   // batched plans use the batched / grouped calls
  return verify_impl(plan, A, lda, transA, B, ldb, transB, dtype, partials, r, s, tol, lhs, rhs, scale,
                     accept, BatchLayout{}, hip_stream);
}

extern "C" int cleave_verify_reduce(cleave_plan* plan, const void* A, int64_t lda, int transA,
                                    const void* B, int64_t ldb, int transB, int dtype,
                                    const float* partials, const float* r, const float* s, double tol,
                                    double* lhs, double* rhs, double* scale, int32_t* accept,
                                    void* C, int64_t ldc, int out_dtype, void* hip_stream) {
  if (!plan || plan->batch > 0 || !C) return CLEAVE_EINVAL;
  if (out_dtype != CLEAVE_F32 && out_dtype != CLEAVE_BF16) return CLEAVE_EINVAL;
  if (ldc < plan->N || !aligned(C, out_dtype == CLEAVE_BF16 ? 2 : 4)) return CLEAVE_EINVAL;
  int rc = ensure_verify_tables_host(plan);
  if (rc != CLEAVE_OK) return rc;
  if (plan->verify->max_ksplit > static_cast<uint32_t>(cleave::kMaxFusedSplits)) {
    // more splits per tile than the fused pass carries: the two passes one after the other
    rc = verify_impl(plan, A, lda, transA, B, ldb, transB, dtype, partials, r, s, tol, lhs, rhs, scale,
                     accept, BatchLayout{}, hip_stream);
    if (rc != CLEAVE_OK) return rc;
    return reduce_impl(plan, partials, C, ldc, out_dtype, BatchLayout{}, hip_stream);
  }
  AggregateTarget agg;
  agg.C = C;
  agg.ldc = ldc;
  agg.out_dtype = out_dtype;
  return verify_impl(plan, A, lda, transA, B, ldb, transB, dtype, partials, r, s, tol, lhs, rhs, scale,
                     accept, BatchLayout{}, hip_stream, agg);
}

extern "C" int cleave_verify_batched(cleave_plan* plan, const void* A, int64_t lda, int transA,
                                     int64_t a_outer, int64_t a_inner, const void* B, int64_t ldb,
                                     int transB, int64_t b_outer, int64_t b_inner, int64_t n_inner,
                                     int dtype, const float* partials, const float* r, const float* s,
                                     double tol, double* lhs, double* rhs, double* scale,
                                     int32_t* accept, void* hip_stream) {
  if (!plan || plan->batch < 1) return CLEAVE_EINVAL;
  if (n_inner < 1 || n_inner > std::numeric_limits<uint32_t>::max() || plan->batch % n_inner != 0)
    return CLEAVE_EINVAL;
  if (a_outer < 0 || a_inner < 0 || b_outer < 0 || b_inner < 0) return CLEAVE_EINVAL;
  return verify_impl(plan, A, lda, transA, B, ldb, transB, dtype, partials, r, s, tol, lhs, rhs, scale,
                     accept, strided_layout(n_inner, a_outer, a_inner, b_outer, b_inner, 0, 0), hip_stream);
}

extern "C" int cleave_verify_grouped(cleave_plan* plan, int64_t n_members, const void* const* A_list,
                                     int64_t lda, int transA, const void* const* B_list, int64_t ldb,
                                     int transB, int dtype, const float* partials, const float* r,
                                     const float* s, double tol, double* lhs, double* rhs,
                                     double* scale, int32_t* accept, void* hip_stream) {
  if (!plan || plan->batch < 1 || plan->batch > cleave::kMaxGroup || n_members != plan->batch)
    return CLEAVE_EINVAL;
  if (dtype != CLEAVE_F32 && dtype != CLEAVE_BF16) return CLEAVE_EINVAL;
  const int eb = dtype == CLEAVE_BF16 ? 2 : 4;
  BatchLayout bl;
  bl.shape.n_group = static_cast<uint32_t>(plan->batch);
  const void* A = nullptr;
  const void* B = nullptr;
  int rc = group_offsets(A_list, plan->batch, eb, &bl.a, &A);
  if (rc != CLEAVE_OK) return rc;
  rc = group_offsets(B_list, plan->batch, eb, &bl.b, &B);
  if (rc != CLEAVE_OK) return rc;
  return verify_impl(plan, A, lda, transA, B, ldb, transB, dtype, partials, r, s, tol, lhs, rhs, scale,
                     accept, bl, hip_stream);
}
