// Where a work item's accumulators go, and the stores that put them there;
// shared by the two execute kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "bf16_round.h"
#include "kernels.h"
#include "load_record.h"

namespace cleave {

typedef float tile_f32x16 __attribute__((ext_vector_type(16)));
typedef float tile_f32x4 __attribute__((ext_vector_type(4)));

// Destination of one sub-tile: element (0, 0) of the sub-tile and the row
// stride in elements (the element type is a property of the launch:
// ExecuteArgs::c_bf16).
struct TileTarget {
  unsigned char* base;
  int64_t ld;
  bool stream;
};

// Partial mode (args.C == nullptr): the benchmark's fp32 block, row-major
// m_len x n_len at partial_off (paper Sec. 4.1: a device returns its
// alpha x beta block).  Assemble mode: the block's place in the output matrix
// itself (Sec. 3.2: the PS assembles the returned blocks) -- only meaningful
// for tasks that cover the whole inner dimension.
__device__ __forceinline__ TileTarget tile_target(const ExecuteArgs& args, const WorkItem& w) {
  TileTarget t;
  t.stream = w.k0 < args.stream_below_k;
  if (args.C == nullptr) {
    t.ld = w.out_ld;
    t.base = reinterpret_cast<unsigned char*>(args.partials + w.out_off);
  } else {
    t.ld = args.ldc;
    const int64_t off = member_offset(args.c_at, args.batch, w.gemm_id) +
                        static_cast<int64_t>(w.m_base) * t.ld + w.n_base;
    t.base = static_cast<unsigned char*>(args.C) + off * (args.c_bf16 ? 2 : 4);
  }
  return t;
}

// Stores a wave's MB x NB grid of 32 x 32 MFMA accumulator blocks.  A block
// leaves lane l with column l % 32 and rows 8*q + 4*(l / 32) + r, so half a
// wave writes one aligned run of 32 elements per store.  row0 / col0: this
// lane's first row and column inside the sub-tile; one per-thread base pointer
// plus wave-uniform row offsets keeps the stores free of address arithmetic.
// `interior`: the sub-tile is full, no bounds checks.  Plain stores, whatever the
// output's size: with outputs that the caches hold, non-temporal ones made execute ~1 %
// faster and the reducer that follows ~10 % slower; with larger ones, where store_rows
// streams, they were not measured for the kernel that uses this.
template <int MB, int NB, typename T, typename Cvt>
__device__ __forceinline__ void store_blocks(const tile_f32x16 (&acc)[MB][NB], T* tp, int64_t ld,
                                             int row0, int col0, int m_valid, int n_valid,
                                             bool interior, Cvt cvt) {
  if (interior) {
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          T* p = tp + static_cast<int64_t>(i * 32 + q * 8 + r) * ld;
#pragma unroll
          for (int j = 0; j < NB; ++j) p[j * 32] = cvt(acc[i][j][q * 4 + r]);
        }
  } else {
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int rr = i * 32 + q * 8 + r;
          T* p = tp + static_cast<int64_t>(rr) * ld;
#pragma unroll
          for (int j = 0; j < NB; ++j)
            if (row0 + rr < m_valid && col0 + j * 32 < n_valid) p[j * 32] = cvt(acc[i][j][q * 4 + r]);
        }
  }
}

// Stores a wave's MB x NB grid of 16 x 16 blocks of which a lane has row
// lane % 16 and columns 4 (lane / 16) .. + 3.  One row of blocks at a time is
// turned through a row-major image in LDS that belongs to this wave alone
// (`image`), so that neighbouring lanes leave with neighbouring 16 bytes of a
// row and a store instruction writes whole 128-byte lines in lane order (64-byte
// rows for bf16 and two blocks).  The order counts: the same lines written by
// lanes eight apart (the lanes' own 16 bytes, pairs of blocks exchanged across
// lanes without LDS), or as the 64-byte rows of one block at a time, make every
// group of sixteen lanes touch eight or sixteen lines: 128 products of 1024 x
// 1024 x 128 into bf16 88 us through the image, 100 without; 16384 x 13824 x
// 5120 in 8 splits 2.41 / 2.68 ms.
//
// wave_row0 / wave_col0: first row and column of the wave's part of the
// sub-tile, of which m_valid x n_valid elements exist (n_valid a multiple of 8).
// The target may have any alignment of its elements.  LDS executes a wave's
// accesses in issue order, and the compiler is kept from reordering them by the
// asm statements; no other wave touches the image, so no barrier is involved.
constexpr int kBlockImageBytes = 16 * 64 * 4;
//
// STREAM: non-temporal stores, for outputs that the caches cannot hold until they
// are read (ExecuteArgs::stream_below_k).  The differing asm statements keep the
// compiler from merging this form with the other one, which would drop the hint.
template <bool BF16, bool INTERIOR, bool STREAM, int MB, int NB>
__device__ __forceinline__ void store_rows(const tile_f32x4 (&acc)[MB][NB], const TileTarget& t, unsigned char* image,
                                           int wave_row0, int wave_col0, int lane, int m_valid, int n_valid) {
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(2)));
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  constexpr int EB = BF16 ? 2 : 4;             // bytes per element
  constexpr int Q = NB * EB;                   // 16-byte pieces of an image row
  constexpr int R = 16 / Q;                    // image rows in a cycle of the banks
  constexpr int RR = 64 / Q;                   // rows per read of the whole wave
  static_assert(16 * Q * 16 <= kBlockImageBytes && Q * R == 16, "image");
  // piece q of row r sits at r * Q + (q ^ (r / R % Q)): a write's rows and a
  // read's pieces both fall into different banks
  const int wrow = lane & 15, wflip = (wrow / R) & (Q - 1);
  const int rrow = lane / Q, rpiece = lane % Q;
  const int row = wave_row0 + rrow, col = wave_col0 + rpiece * (16 / EB);
  unsigned char* gp = t.base + (row * t.ld + col) * EB;
  const int64_t pitch = t.ld * EB;
#pragma unroll
  for (int i = 0; i < MB; ++i, gp += 16 * pitch) {
    if constexpr (STREAM) asm volatile("; streamed" ::: "memory");
    else asm volatile("" ::: "memory");
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      if constexpr (BF16) {
        const int piece = (2 * j + (lane >> 5)) ^ wflip;
        *reinterpret_cast<u32x2*>(image + (wrow * Q + piece) * 16 + 8 * ((lane >> 4) & 1)) =
            u32x2{pack_bf16(acc[i][j][0], acc[i][j][1]), pack_bf16(acc[i][j][2], acc[i][j][3])};
      } else {
        *reinterpret_cast<tile_f32x4*>(image + (wrow * Q + ((4 * j + (lane >> 4)) ^ wflip)) * 16) = acc[i][j];
      }
    }
    asm volatile("" ::: "memory");
    u32x4 v[16 / RR];
#pragma unroll
    for (int k = 0; k < 16 / RR; ++k) {
      const int r = rrow + RR * k;
      v[k] = *reinterpret_cast<const u32x4*>(image + (r * Q + (rpiece ^ ((r / R) & (Q - 1)))) * 16);
    }
    asm volatile("" ::: "memory");
#pragma unroll
    for (int k = 0; k < 16 / RR; ++k)
      if (INTERIOR || (row + i * 16 + RR * k < m_valid && col < n_valid)) {
        u32x4_any* const to = reinterpret_cast<u32x4_any*>(gp + RR * k * pitch);
        if constexpr (STREAM) __builtin_nontemporal_store(v[k], to);
        else *to = v[k];
      }
  }
  if constexpr (STREAM) asm volatile("; end of streamed stores" ::: "memory");
}

// One 16 x 16 block: lane l has column l % 16 and rows 4 (l / 16) .. + 3.
__device__ __forceinline__ void store_block(tile_f32x4 acc, const TileTarget& t, bool bf16, int row0, int col0,
                                            int m_valid, int n_valid) {
  if (col0 >= n_valid) return;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    if (row0 + r >= m_valid) break;
    const int64_t at = (row0 + r) * t.ld + col0;
    if (bf16) reinterpret_cast<uint16_t*>(t.base)[at] = to_bf16_bits(acc[r]);
    else reinterpret_cast<float*>(t.base)[at] = acc[r];
  }
}

template <int MB, int NB>
__device__ __forceinline__ void store_tile(const tile_f32x16 (&acc)[MB][NB], const TileTarget& t,
                                           bool bf16, int row0, int col0, int m_valid,
                                           int n_valid, bool interior) {
  if (!bf16) {
    float* tp = reinterpret_cast<float*>(t.base) + row0 * t.ld + col0;
    store_blocks<MB, NB>(acc, tp, t.ld, row0, col0, m_valid, n_valid, interior,
                         [](float x) { return x; });
  } else {
    uint16_t* tp = reinterpret_cast<uint16_t*>(t.base) + row0 * t.ld + col0;
    store_blocks<MB, NB>(acc, tp, t.ld, row0, col0, m_valid, n_valid, interior,
                         [](float x) { return to_bf16_bits(x); });
  }
}

}  // namespace cleave
