// Launch tables that are written on the device: the work-item lists of subset
// launches and the aggregation's records.
//
// A re-issued subset (paper Sec. 4.2, churn recovery: the unfinished shards of
// a departed device are dispatched again) is a list of task indices.  The host
// decides where each task's work items go; this kernel derives the items from
// the task records already on the device.  The (task, destination) pairs come
// in through the kernel arguments.
#include <hip/hip_runtime.h>

#include "kernels.h"
#include "plan_internal.h"

namespace cleave {

namespace {

// One wave per entry; lane l writes sub-tiles l, l + 64, ...
__global__ __launch_bounds__(64) void expand_subset_kernel(ExpandArgs args) {
  const uint32_t e = blockIdx.x;
  if (e >= args.n_entries) return;
  const SubsetEntry entry = args.entries[e];
  const cleave_task t = args.tasks[entry.task];
  const SubTiling s = sub_tiling(t, args.fine != 0);
  for (uint32_t sub = threadIdx.x; sub < s.count(); sub += 64)
    args.out[entry.dst + sub] = make_work_item(t, entry.task, s, sub);
}

// One workgroup per tile at a time; its threads write one run's record each.
constexpr int kTileThreads = 256;
__global__ __launch_bounds__(kTileThreads) void expand_reduce_kernel(const cleave_task* tasks, const ReduceTile* tiles,
                                                                     int64_t n_tiles, ReduceItem* out) {
  for (int64_t i = blockIdx.x; i < n_tiles; i += gridDim.x) {
    const ReduceTile tile = tiles[i];
    const cleave_task t = tasks[tile.task];
    const uint64_t block = static_cast<uint64_t>(t.m_len) * t.n_len;
    const uint64_t runs = (block + tile.run - 1) / tile.run;
    for (uint64_t r = threadIdx.x; r < runs; r += kTileThreads)
      out[tile.first + r] = make_reduce_item(t, r * tile.run, tile.run);
  }
}

}  // namespace

hipError_t launch_expand_reduce(const cleave_task* tasks, const ReduceTile* tiles, int64_t n_tiles, ReduceItem* out,
                                hipStream_t stream) {
  if (n_tiles == 0) return hipSuccess;
  const int grid = static_cast<int>(n_tiles < (1 << 16) ? n_tiles : 1 << 16);
  hipLaunchKernelGGL(expand_reduce_kernel, dim3(grid), dim3(kTileThreads), 0, stream, tasks, tiles, n_tiles, out);
  return hipGetLastError();
}

hipError_t launch_expand_subset(const ExpandArgs& args, hipStream_t stream) {
  if (args.n_entries == 0) return hipSuccess;
  hipLaunchKernelGGL(expand_subset_kernel, dim3(args.n_entries), dim3(64), 0, stream, args);
  return hipGetLastError();
}

}  // namespace cleave
