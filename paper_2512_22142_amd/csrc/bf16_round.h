// fp32 -> bf16 on the GPU.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace cleave {

// Two values rounded to nearest even, `lo` in the low half: one instruction of
// gfx950 (v_cvt_pk_bf16_f32) where the integer form takes six per value.  Same
// bits as that form for all 2^32 inputs (compared by the tests): subnormals are
// kept, NaN stays a quiet NaN with the upper bits of its payload.
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{lo, hi}), bf16x2));
}

__device__ __forceinline__ uint16_t to_bf16_bits(float x) {
  return __builtin_bit_cast(uint16_t, static_cast<__bf16>(x));
}

}  // namespace cleave
