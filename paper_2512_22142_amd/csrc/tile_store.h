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

// Destination of one sub-tile: element (0, 0) of the sub-tile and the row
// stride in elements (the element type is a property of the launch:
// ExecuteArgs::c_bf16).
struct TileTarget {
  unsigned char* base;
  int64_t ld;
};

// Partial mode (args.C == nullptr): the benchmark's fp32 block, row-major
// m_len x n_len at partial_off (paper Sec. 4.1: a device returns its
// alpha x beta block).  Assemble mode: the block's place in the output matrix
// itself (Sec. 3.2: the PS assembles the returned blocks) -- only meaningful
// for tasks that cover the whole inner dimension.
__device__ __forceinline__ TileTarget tile_target(const ExecuteArgs& args, const WorkItem& w) {
  TileTarget t;
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
// `interior`: the sub-tile is full, no bounds checks.  Plain stores:
// non-temporal ones make execute ~1 % faster but the reducer that follows
// ~10 % slower.
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

// A full sub-tile, turned through a 4 KB row-major image
// in LDS that belongs to this wave alone (`image`), so that a lane leaves with
// 16 consecutive bytes of one row and a store instruction writes eight whole
// 128-byte lines instead of 64 elements in two rows.  The image holds one
// 32 x 32 block of fp32 or two neighbouring ones of bf16 (32 rows x 64
// columns), which therefore take half the LDS traffic and store instructions.
// The values and their addresses are those of store_blocks.  wave_row0 /
// wave_col0: first row and column of the wave's part of the sub-tile.  The
// target must allow 16-byte (fp32) or 8-byte (bf16) stores at every fourth
// column.  LDS executes a wave's accesses in issue order, and the compiler is
// kept from reordering them by the asm statements; no other wave touches the
// image, so no barrier is involved.
//
// bf16 values are rounded where they are, two rows of a column per
// instruction; one lane exchange then turns the pairs of two neighbouring
// columns round, so that a lane writes two neighbouring columns of one row as
// one dword.  (128 products of 1024 x 1024 x 128 into bf16 followed by 128 of
// 1024 x 128 x 1024 into fp32: 182 us; 200 us with the rounding on the way out
// of the image, four values per lane in integer arithmetic, and 8-byte stores,
// where the store phase is the longer half of a work item of two K steps.)
constexpr int kBlockImageBytes = 32 * 32 * 4;
template <int NB, bool BF16>
__device__ __forceinline__ constexpr int staged_stores_per_block_row() {
  return NB * (BF16 ? 2 : 4);
}

template <int MB, int NB>
__device__ __forceinline__ void store_tile_staged_f32(const tile_f32x16 (&acc)[MB][NB],
                                                           const TileTarget& t, unsigned char* image,
                                                           int wave_row0, int wave_col0, int lane) {
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  float* wr = reinterpret_cast<float*>(image) + (4 * (lane >> 5)) * 32 + (lane & 31);
  const f32x4* rd = reinterpret_cast<const f32x4*>(image) + lane;   // row lane / 8 (+ 8 k), columns 4 (lane % 8) ..
  float* gp = reinterpret_cast<float*>(t.base) + static_cast<int64_t>(wave_row0 + (lane >> 3)) * t.ld + wave_col0 +
              (lane & 7) * 4;
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      asm volatile("" ::: "memory");
#pragma unroll
      for (int r = 0; r < 16; ++r) wr[((r >> 2) * 8 + (r & 3)) * 32] = acc[i][j][r];
      asm volatile("" ::: "memory");
      f32x4 v[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = rd[64 * k];
      asm volatile("" ::: "memory");
#pragma unroll
      for (int k = 0; k < 4; ++k)
        *reinterpret_cast<f32x4*>(gp + static_cast<int64_t>(i * 32 + 8 * k) * t.ld + j * 32) = v[k];
    }
}

template <int MB, int NB>
__device__ __forceinline__ void store_tile_staged_bf16(const tile_f32x16 (&acc)[MB][NB],
                                                       const TileTarget& t, unsigned char* image,
                                                       int wave_row0, int wave_col0, int lane) {
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  typedef uint32_t u32x4_at8 __attribute__((ext_vector_type(4), aligned(8)));   // rows start on 8 bytes
  constexpr int W = NB % 2 == 0 ? 2 : 1;      // blocks side by side in the image
  constexpr int RW = 16 * W;                  // dwords of an image row
  constexpr int QR = RW / 4;                  // 16-byte pieces of an image row
  constexpr int RR = 64 / QR;                 // rows per read of the whole wave
  // An even lane writes columns (l32, l32 + 1) of its rows 8 q + 4 lh + 2 p, an
  // odd lane columns (l32 - 1, l32) of the rows behind them.  The two halves of
  // a wave are four rows apart, which is the same banks: with two blocks, rows
  // with bit 2 set are kept with their 16-dword halves exchanged.
  const int lh = lane >> 5, odd = lane & 1;
  const uint32_t select = odd ? 0x03020706u : 0x05040100u;   // (other high, own high) : (own low, other low)
  uint32_t* wr = reinterpret_cast<uint32_t*>(image) + (4 * lh + odd) * RW + ((lane & 31) >> 1);
  uint32_t* wr_half[2] = {wr + (W == 2 ? 16 * lh : 0), wr + 16 * (1 - lh)};
  const int row = lane / QR, quad = (lane % QR) ^ (W == 2 ? 4 * ((row >> 2) & 1) : 0);
  const u32x4* rd = reinterpret_cast<const u32x4*>(image) + row * QR + quad;
  uint16_t* gp = reinterpret_cast<uint16_t*>(t.base) + static_cast<int64_t>(wave_row0 + row) * t.ld + wave_col0 +
                 (lane % QR) * 8;
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; j += W) {
      asm volatile("" ::: "memory");
#pragma unroll
      for (int h = 0; h < W; ++h)
#pragma unroll
        for (int p = 0; p < 8; ++p) {   // rows 8 * (p / 2) + 4 lh + 2 * (p % 2), and the next
          const uint32_t own = pack_bf16(acc[i][j + h][2 * p], acc[i][j + h][2 * p + 1]);
          const uint32_t other = __builtin_amdgcn_update_dpp(0u, own, 0xB1, 0xF, 0xF, true);   // lane ^ 1
          wr_half[h][(8 * (p >> 1) + 2 * (p & 1)) * RW] = __builtin_amdgcn_perm(other, own, select);
        }
      asm volatile("" ::: "memory");
      u32x4 v[32 / RR];
#pragma unroll
      for (int k = 0; k < 32 / RR; ++k) v[k] = rd[64 * k];
      asm volatile("" ::: "memory");
#pragma unroll
      for (int k = 0; k < 32 / RR; ++k)
        *reinterpret_cast<u32x4_at8*>(gp + static_cast<int64_t>(i * 32 + RR * k) * t.ld + j * 32) = v[k];
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
