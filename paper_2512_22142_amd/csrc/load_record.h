// Launch-table records into scalar registers.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "plan_internal.h"

namespace cleave {

// Record `idx` (48 bytes, 16-byte aligned) of a table that the kernel reading it
// does not write (a kernel launched before it may have): read through the constant address space, a wave-uniform address becomes scalar
// loads whose completion the compiler tracks, even though the kernels also store
// to global memory.
template <typename Record>
__device__ __forceinline__ Record load_record(const Record* table, int64_t idx) {
  static_assert(sizeof(Record) == 48, "three 16-byte words");
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  typedef const __attribute__((address_space(4))) u32x4* const_words;
  const_words src = (const_words)(table + idx);
  uint32_t words[12];
#pragma unroll
  for (int v = 0; v < 3; ++v) {
    const u32x4 q = src[v];
#pragma unroll
    for (int e = 0; e < 4; ++e) words[4 * v + e] = q[e];
  }
  Record r;
  __builtin_memcpy(&r, words, sizeof(r));
  return r;
}

__device__ __forceinline__ WorkItem load_work_item(const WorkItem* items, int64_t idx) {
  return load_record(items, idx);
}

}  // namespace cleave
