// Sub-GEMM task executor for gfx950 (paper Sec. 4.1: a task multiplies its
// rows of A with its columns of B; here restricted to its chunk of the inner
// dimension, and the fp32 partial block goes to the task's slot in HBM).
//
// This is the general executor: fp32 inputs, and every bf16 work item that the
// direct-to-LDS kernel does not take (operands whose rows do not start on
// 16-byte boundaries, chunks or tile rows that are no whole eights where the
// operand runs along them, rows longer than its 32-bit offsets).  One workgroup computes one TM x TN part of a work
// item over the task's whole chunk [k0, k0 + k_len), in ascending steps of 128
// bytes of K per row (64 bf16 / 32 fp32 elements) and, inside a step, in
// ascending 32-byte sub-steps; the order of the MFMA accumulation for an
// output element therefore depends only on the task record (and is the direct
// kernel's), which is what makes a re-issued task bitwise reproducible.
//
// Data path per K step: global -> VGPR in 16-byte loads -> LDS -> fragments ->
// MFMA 32x32x16 bf16 (or 32x32x2 fp32, 16x16x4 in the smallest tile) into fp32
// accumulators.
//   * The loads need only the alignment of an element (global memory takes
//     16-byte loads at any address), so an odd leading dimension or chunk
//     start costs a second cache line per row, not sixteen-fold instructions.
//     Elements beyond the chunk must be zero and loads must stay inside the
//     operand, so the steps that touch an end (the last of a chunk) load the
//     last 16 bytes that are inside and shift the wanted elements down.
//   * Loads run SETS steps ahead in registers and LDS holds two steps, with one
//     barrier per step: what bounds a launch with few workgroups is the latency
//     of a step's loads, and SETS of them overlap.  Where a wave is nearly alone on its
//     SIMD (kAhead) fragments are read a step before they are multiplied: LDS is written
//     two steps ahead then, and loads run four ahead.
//     The waits on them count loads in flight, so the loads of a step past the
//     last one are issued too (one line, already read) rather than skipped.
//   * An operand whose rows hold less than 16 bytes is loaded one element at a
//     time; the other operand, which is the large one then, still takes 16-byte
//     loads.  With both by element and the guards per element (the loads of a
//     chunk one behind the other, registers spilled) outputs one to seven
//     columns wide took up to 1.3 times the 128 x 128 element tile that this one
//     replaced: us, that tile / both by element / now, bf16 131072 x 1 x 512
//     161 / 206 / 56, 64 x 1 x 4096 159 / 172 / 51, fp32 1 x 131072 x 512 with
//     K x M and K x N operands 168 / 201 / 143.
//   * LDS images are of the direct kernel's kinds (swizzled K-contiguous rows; k
//     rows read through the LDS transpose read for bf16, one dword per k for
//     fp32), so nothing is transposed in registers.
//
// What bounds it: fp32, the matrix cores (64 cycles per 32x32x2): 4096^3 as
// 512 x 512 x 1024 tasks runs at 142 TFLOP/s of 157 nominal.  bf16, the LDS (32 x 64
// wave tiles read 192 bytes per clock and CU at full MFMA rate, and the tile's
// refill comes on top): the same with an odd leading dimension 620-640 TFLOP/s.
// Execute + reduce against unaligned operands loaded by element, and one fp32 tile
// of 256 x 256 or 128 x 128 with one step in flight: forward, dX and dW of 3001 x 1000
// x 2500 bf16 in 4 splits 155 / 1173 us, of 2048 x 768 x 3072 fp32 255 / 403 us, 512^3
// fp32 10.3 / 26.7 us (of the last, 4.5 us are host time saved by the native argument
// checks).
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "plan_internal.h"
#include "kernels.h"
#include "tile_store.h"

namespace cleave {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4* lds_s16x4;
// 16 bytes at an address that is only a multiple of an element
typedef uint32_t u32x4_at2 __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t u32x4_at4 __attribute__((ext_vector_type(4), aligned(4)));

template <int V>
using int_c = std::integral_constant<int, V>;

// Kernel shape: element bytes, workgroup tile TM x TN computed by WM x WN
// waves, SETS register sets of loads in flight, WPE waves per SIMD.
template <int EB_, int TM_, int TN_, int WM_, int WN_, int SETS_, int WPE_>
struct Shape {
  static constexpr int EB = EB_, TM = TM_, TN = TN_, WM = WM_, WN = WN_, SETS = SETS_, WPE = WPE_;
  static constexpr int NT = WM * WN * 64;
  static constexpr int E = 16 / EB;             // elements per 16-byte chunk
  static constexpr int KS = 128 / EB;           // elements of K per step
  static constexpr int WTM = TM / WM, WTN = TN / WN;
  // MFMA block: 32 x 32 (x 2, or 16 for bf16), or, fp32 wave tiles of one, 16 x 16 (x 4)
  static constexpr int BLK = WTM < 32 ? 16 : 32;
  static constexpr int MB = WTM / BLK, NB = WTN / BLK;
  static constexpr int kSub = 4;                // 32-byte sub-steps per step
  static constexpr int kATile = TM * 128, kBTile = TN * 128;   // bytes
  static constexpr int kStage = kATile + kBTile;
  // the fragments of the next K step are read while a step is multiplied
  static constexpr bool kAhead = SETS == 2 && MB == 1 && NB == 1 && (BLK == 16 || WPE == 2);
  static_assert(BLK == 32 || (EB == 4 && MB == 1 && NB == 1), "16 x 16: one block per wave, fp32");
  static_assert(SETS == 1 || SETS == 2, "register sets rotate with the two LDS stages");
};

// All LDS accesses of this wave are done; then the workgroup barrier.  Loads
// to registers stay in flight across it.
#define CLEAVE_LDS_BARRIER() asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory")

// The elements of a 16-byte chunk moved down by `shift` elements, zeros above
// (shift >= E: all zero).
template <int EB>
__device__ __forceinline__ u32x4 shift_down(u32x4 v, int shift) {
  constexpr int E = 16 / EB;
  const int bits = shift * EB * 8;
  const uint64_t lo = v[0] | (static_cast<uint64_t>(v[1]) << 32);
  const uint64_t hi = v[2] | (static_cast<uint64_t>(v[3]) << 32);
  const uint64_t across = bits == 0 ? 0 : hi << ((64 - bits) & 63);
  uint64_t l = bits < 64 ? (lo >> (bits & 63)) | across : hi >> ((bits - 64) & 63);
  uint64_t h = bits < 64 ? hi >> (bits & 63) : 0;
  if (shift >= E) l = h = 0;
  return u32x4{static_cast<uint32_t>(l), static_cast<uint32_t>(l >> 32), static_cast<uint32_t>(h),
               static_cast<uint32_t>(h >> 32)};
}

// ---------------------------------------------------------------------------
// Operand tile: R rows (an m or n index) x 128 bytes of K, moved global ->
// registers -> LDS by NT threads, NV 16-byte chunks each.  Slot s of the LDS
// image is written by thread s % NT.
//   KCONTIG: tile rows of 128 bytes, slot = r * 8 + (chunk ^ ((r >> 1) & 7)).
//   else:    KS k rows of R elements, slot = k * CH + (chunk ^ swizzle(k)); the
//            swizzle spreads over the banks the four k rows of a transpose
//            read (bf16) or the k rows of the two halves of a wave (fp32).
// ---------------------------------------------------------------------------
template <int EB, int R, int NT, bool KCONTIG, bool ELEMENTWISE>
struct OperandTile {
  static_assert(KCONTIG || !ELEMENTWISE, "element loads fill the K-contiguous image, whatever the storage");
  static constexpr int E = 16 / EB;
  static constexpr int KS = 128 / EB;
  static constexpr int CH = R / E;                  // chunks per k row
  static constexpr int NV = R * 8 / NT;
  static_assert(R * 8 % NT == 0, "tile / thread count");

  static __device__ __forceinline__ int k_swizzle(int k) {
    if constexpr (EB == 4) return (CH == 8 ? 4 : 8) * ((k >> 2) & 1);
    else if constexpr (CH == 8) return 4 * ((k >> 1) & 1);
    else return 4 * (k & 3);
  }
  // (tile row, k) of the first element of this thread's chunk i
  static __device__ __forceinline__ void where(int i, int t, int* r, int* k) {
    const int slot = t + NT * i;
    if constexpr (KCONTIG) {
      *r = slot >> 3;
      *k = ((slot & 7) ^ ((*r >> 1) & 7)) * E;
    } else {
      *k = slot / CH;
      *r = ((slot % CH) ^ k_swizzle(*k)) * E;
    }
  }

  const unsigned char* base;    // element (tile row 0, k0); wave-uniform
  const unsigned char* next;    // where the next step's loads start from; wave-uniform
  uint32_t off[NV];             // byte offset of each chunk from `next`
  int64_t row_stride, k_stride; // bytes
  int r_valid, k_len, steps;
  int left_to_row_end;          // !KCONTIG: elements from tile row 0 to the end of a stored row (>= r_valid)
  int edge_step;                // the step whose loads must be kept inside the operand (-1: none)

  // k0: chunk start; k_total, r_total: extent of the operand; r0: tile row 0.
  __device__ __forceinline__ void init(const unsigned char* b, int64_t rs, int64_t ks, int rv, int64_t r0,
                                       int64_t r_total, int64_t k0, int len, int64_t k_total, int t) {
    base = next = b;
    row_stride = rs * EB;
    k_stride = ks * EB;
    r_valid = rv;
    k_len = len;
    steps = chunk_steps(len, KS);
    edge_step = len % KS ? steps - 1 : -1;
    if constexpr (KCONTIG) {
      left_to_row_end = 0;
    } else {
      const int64_t left = r_total - r0;
      left_to_row_end = static_cast<int>(left < 2 * R ? left : 2 * R);
      // a chunk that runs past the end of a stored row stays inside the operand
      // except on the operand's last row
      const bool past_end = (rv + E - 1) / E * E > left_to_row_end;
      if (past_end && k0 + len == k_total) edge_step = steps - 1;
    }
    if constexpr (ELEMENTWISE) return;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      int r, k;
      where(i, t, &r, &k);
      // rows beyond the valid ones feed outputs that are never stored: any row of the tile will do
      if constexpr (KCONTIG) r = min(r, rv - 1);
      else r = r < rv ? r : 0;
      off[i] = static_cast<uint32_t>(r * row_stride + k * k_stride);
    }
  }

  // Chunk i of the edge step is loaded `shift` elements before the wanted
  // element, so that the 16 bytes end inside the row (K-contiguous: inside the
  // chunk, everything behind it being zero).  Returns the byte offset from 16
  // bytes before the step's start.
  __device__ __forceinline__ uint32_t edge_source(int i, int t, int* shift) const {
    int r, k;
    where(i, t, &r, &k);
    const int k_left = k_len - edge_step * KS;    // 1 .. KS
    int at;
    int64_t row;
    if constexpr (KCONTIG) {
      row = min(r, r_valid - 1) * row_stride;
      at = min(k, k_left - E);                    // > -E, and the row holds E elements up to the chunk's end
      *shift = k - at;
    } else {
      row = min(k, k_left - 1) * k_stride;
      r = r < r_valid ? r : 0;
      at = min(r, left_to_row_end - E);           // > -E, and a stored row holds E elements
      *shift = k < k_left ? r - at : E;
    }
    return static_cast<uint32_t>(row + (at + E) * EB);
  }

  // One element at a time, for operands whose stored rows hold less than a
  // chunk (or end less than a chunk behind their start) and for rows too long
  // for 32-bit offsets.  Elements beyond the chunk repeat the address of its
  // last one and are dropped, so that a chunk's loads are in flight together.
  __device__ __forceinline__ void load_elements(u32x4 (&v)[NV], int s, int t) const {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      int r, k;
      where(i, t, &r, &k);
      const uint32_t at = static_cast<uint32_t>(k) + static_cast<uint32_t>(s) * KS;   // may pass 2^31
      u32x4 w = {0, 0, 0, 0};
      if (r < r_valid) {
        const int left = static_cast<int>(static_cast<uint32_t>(k_len) - at);
        const unsigned char* q = base + r * row_stride + min(at, static_cast<uint32_t>(k_len - 1)) * k_stride;
#pragma unroll
        for (int e = 0; e < E; ++e) {
          uint32_t x;
          if constexpr (EB == 4) x = *reinterpret_cast<const uint32_t*>(q);
          else x = *reinterpret_cast<const uint16_t*>(q);
          w[e * EB / 4] |= e < left ? x << (e * EB % 4 * 8) : 0u;
          q += e + 1 < left ? k_stride : 0;
        }
      }
      v[i] = w;
    }
  }

  // Steps are loaded in ascending order, each once.  The number of loads in
  // flight must not depend on the control flow (the compiler's waits count
  // them), so a step past the last one is loaded too: one line, already read.
  __device__ __forceinline__ void load(u32x4 (&v)[NV], int s, int t) {
    if constexpr (ELEMENTWISE) {
      load_elements(v, s, t);
      return;
    }
    typedef typename std::conditional<EB == 2, u32x4_at2, u32x4_at4>::type chunk_t;
    if (s == edge_step) {
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        int shift;
        off[i] = edge_source(i, t, &shift);
        __builtin_amdgcn_sched_barrier(0);
      }
      next = base + s * (k_stride * KS) - 16;
    } else if (s == steps) {
#pragma unroll
      for (int i = 0; i < NV; ++i) off[i] = __builtin_amdgcn_readfirstlane(off[0]);
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) v[i] = *reinterpret_cast<const chunk_t*>(next + off[i]);
    if (s + 1 < steps) next += k_stride * KS;
  }

  // A step before the last one: nothing to keep inside the operand.
  __device__ __forceinline__ void load_inner(u32x4 (&v)[NV]) {
    typedef typename std::conditional<EB == 2, u32x4_at2, u32x4_at4>::type chunk_t;
#pragma unroll
    for (int i = 0; i < NV; ++i) v[i] = *reinterpret_cast<const chunk_t*>(next + off[i]);
    next += k_stride * KS;
  }

  // Before the edge step is written to LDS: the wanted elements into place.
  __device__ __forceinline__ void settle(u32x4 (&v)[NV], int s, int t) const {
    if (!ELEMENTWISE && s == edge_step) {
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        int shift;
        edge_source(i, t, &shift);
        v[i] = shift_down<EB>(v[i], shift);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }

  static __device__ __forceinline__ void store(const u32x4 (&v)[NV], unsigned char* lds, int t) {
#pragma unroll
    for (int i = 0; i < NV; ++i) *reinterpret_cast<u32x4*>(lds + (t + NT * i) * 16) = v[i];
  }
};

// How an operand is stored and loaded: K-contiguous or tile-row-contiguous rows
// in 16-byte loads, or one element at a time from either (into the
// K-contiguous image).
enum Storage : int { kByK = 0, kByRow = 1, kElements = 2 };

template <typename S, Storage A, Storage B>
__global__ __launch_bounds__(S::NT, S::WPE) void execute_kernel(ExecuteArgs args) {
  constexpr int EB = S::EB, TM = S::TM, TN = S::TN, MB = S::MB, NB = S::NB, E = S::E, SETS = S::SETS;
  constexpr bool A_K = A != kByRow, B_K = B != kByRow;

  extern __shared__ __align__(16) unsigned char smem[];

  const int t = threadIdx.x;
  const int lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = wave / S::WN;
  const int wn = wave % S::WN;
  const int l32 = lane & (S::BLK - 1);   // row (column) of an MFMA block
  const int lh = S::BLK == 32 ? lane >> 5 : (lane >> 4) & 1;
  const int l4 = lane >> 5;              // 16 x 16 blocks: which of two neighbouring k

  // Lane-constant fragment addresses inside a stage: K-contiguous operands one
  // per sub-step (blocks are 32 rows apart), others one per block.
  const int i16 = lane & 15, kq = i16 >> 2, cq = i16 & 3, nsub = (lane >> 4) & 1;
  const auto frag_addr = [&](int row0, int x, int r_tile, bool kcontig) -> uint32_t {
    if (kcontig) return (row0 + l32) * 128 + (((2 * x + lh) ^ ((l32 >> 1) & 7)) * 16) + (S::BLK == 16 ? 4 * l4 + 8 * lh : 0);
    if (S::BLK == 16) return ((4 * lh + l4) * r_tile + ((row0 + l32) ^ (16 * lh))) * 4;
    if (EB == 4) return (4 * lh * r_tile + ((row0 + x * 32 + l32) ^ (32 * lh))) * 4;
    const int ch = r_tile / 8;
    const int k = 8 * lh + kq;
    const int c = row0 / 8 + x * 4 + 2 * nsub + (cq >> 1);
    const int sw = ch == 8 ? 4 * ((k >> 1) & 1) : 4 * (k & 3);
    return (k * ch + (c ^ sw)) * 16 + (cq & 1) * 8;
  };
  uint32_t a_addr[A_K ? S::kSub : MB], b_addr[B_K ? S::kSub : NB];
#pragma unroll
  for (int x = 0; x < (A_K ? S::kSub : MB); ++x) a_addr[x] = frag_addr(wm * S::WTM, x, TM, A_K);
#pragma unroll
  for (int x = 0; x < (B_K ? S::kSub : NB); ++x) b_addr[x] = S::kATile + frag_addr(wn * S::WTN, x, TN, B_K);

  const int64_t a_rs = args.transA ? 1 : args.lda;
  const int64_t a_ks = args.transA ? args.lda : 1;
  const int64_t b_rs = args.transB ? args.ldb : 1;
  const int64_t b_ks = args.transB ? 1 : args.ldb;

  // Workgroups are dealt round-robin over the XCDs and list position i belongs
  // to XCD i % 8: the parts of an item follow each other on the item's XCD.
  const uint32_t parts = args.parts_m * args.parts_n;
  const uint64_t total = (static_cast<uint64_t>(args.n_items) + 7) / 8 * 8 * parts;
  for (uint64_t b = blockIdx.x; b < total; b += gridDim.x) {
    const uint64_t j = b >> 3;
    const uint64_t it = j / parts * 8 + (b & 7);
    const uint32_t part = static_cast<uint32_t>(j % parts);
    if (it >= static_cast<uint64_t>(args.n_items)) continue;
    const WorkItem item = load_work_item(args.items, static_cast<int64_t>(it));
    const int m_off = static_cast<int>(part / args.parts_n) * TM;
    const int n_off = static_cast<int>(part % args.parts_n) * TN;
    const int m_valid = min(static_cast<int>(item.m_valid) - m_off, TM);
    const int n_valid = min(static_cast<int>(item.n_valid) - n_off, TN);
    if (m_valid <= 0 || n_valid <= 0) continue;
    const int64_t m_base = static_cast<int64_t>(item.m_base) + m_off;
    const int64_t n_base = static_cast<int64_t>(item.n_base) + n_off;
    const int k_len = static_cast<int>(item.k_len);

    OperandTile<EB, TM, S::NT, A_K, A == kElements> ta;
    OperandTile<EB, TN, S::NT, B_K, B == kElements> tb;
    ta.init(static_cast<const unsigned char*>(args.A) +
                (member_offset(args.a_at, args.batch, item.gemm_id) + m_base * a_rs +
                 static_cast<int64_t>(item.k0) * a_ks) * EB,
            a_rs, a_ks, m_valid, m_base, args.M, item.k0, k_len, args.K, t);
    tb.init(static_cast<const unsigned char*>(args.B) +
                (member_offset(args.b_at, args.batch, item.gemm_id) + n_base * b_rs +
                 static_cast<int64_t>(item.k0) * b_ks) * EB,
            b_rs, b_ks, n_valid, n_base, args.N, item.k0, k_len, args.K, t);

    typedef typename std::conditional<S::BLK == 32, f32x16, f32x4>::type block_t;
    block_t acc[MB][NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int jn = 0; jn < NB; ++jn) acc[i][jn] = block_t{};

    u32x4 va[SETS][ta.NV], vb[SETS][tb.NV];
    auto fetch = [&](auto set_tag, int s) {
      constexpr int set = decltype(set_tag)::value;
      ta.load(va[set], s, t);
      tb.load(vb[set], s, t);
    };
    auto commit = [&](auto set_tag, auto stage_tag, int s) {
      constexpr int set = decltype(set_tag)::value, stage = decltype(stage_tag)::value;
      ta.settle(va[set], s, t);
      tb.settle(vb[set], s, t);
      ta.store(va[set], smem + stage * S::kStage, t);
      tb.store(vb[set], smem + stage * S::kStage + S::kATile, t);
    };

    u32x4 fa[2][MB], fb[2][NB];
    auto tr_read = [&](const unsigned char* q) -> u32x2 {
      return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)q));
    };
    auto read_frag = [&](const unsigned char* stage, const uint32_t* addr, auto kcontig_tag, auto rows_tag,
                         auto ks_tag, int x) -> u32x4 {
      constexpr bool KC = decltype(kcontig_tag)::value;
      constexpr int R = decltype(rows_tag)::value, KSUB = decltype(ks_tag)::value;
      if constexpr (S::BLK == 16 && KC) {
        // k of the sub-step: 4 lh + l4, and two further on; half of the lanes read them
        // the other way round (mma puts them back), so that the 64 words are in different banks
        const uint32_t one = *reinterpret_cast<const uint32_t*>(stage + addr[KSUB]);
        const uint32_t two = *reinterpret_cast<const uint32_t*>(stage + (addr[KSUB] ^ 8));
        return u32x4{one, two, 0, 0};
      } else if constexpr (S::BLK == 16) {
        const uint32_t* q = reinterpret_cast<const uint32_t*>(stage + addr[x] + KSUB * (8 * R * 4));
        return u32x4{q[0], q[2 * R], 0, 0};
      } else if constexpr (KC) {
        return *reinterpret_cast<const u32x4*>(stage + addr[KSUB] + x * 32 * 128);
      } else if constexpr (EB == 2) {
        const unsigned char* q = stage + addr[x] + KSUB * (16 * R * 2);
        const u32x2 lo = tr_read(q), hi = tr_read(q + 4 * R * 2);
        return u32x4{lo[0], lo[1], hi[0], hi[1]};
      } else {
        const uint32_t* q = reinterpret_cast<const uint32_t*>(stage + addr[x] + KSUB * (8 * R * 4));
        return u32x4{q[0], q[R], q[2 * R], q[3 * R]};
      }
    };
    auto read_frags = [&](int stage, auto ks_tag, int buf) {
#pragma unroll
      for (int i = 0; i < MB; ++i)
        fa[buf][i] = read_frag(smem + stage * S::kStage, a_addr, std::bool_constant<A_K>{}, int_c<TM>{}, ks_tag, i);
#pragma unroll
      for (int i = 0; i < NB; ++i)
        fb[buf][i] = read_frag(smem + stage * S::kStage, b_addr, std::bool_constant<B_K>{}, int_c<TN>{}, ks_tag, i);
    };
    auto mma = [&](int buf) {
      if constexpr (S::BLK == 16) {
        // One instruction multiplies k, k + 4, k + 1, k + 5 of a sub-step, in this order
        // (lanes 0-15, 16-31, ...): the chain of two 32 x 32 x 2 ones, bit for bit.
        const f32x4 a4 = __builtin_bit_cast(f32x4, A_K && lh ? u32x4{fa[buf][0][1], fa[buf][0][0], 0, 0} : fa[buf][0]);
        const f32x4 b4 = __builtin_bit_cast(f32x4, B_K && lh ? u32x4{fb[buf][0][1], fb[buf][0][0], 0, 0} : fb[buf][0]);
#pragma unroll
        for (int e = 0; e < 2; ++e) acc[0][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a4[e], b4[e], acc[0][0], 0, 0, 0);
      } else if constexpr (EB == 2) {
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int jn = 0; jn < NB; ++jn)
            acc[i][jn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                __builtin_bit_cast(bf16x8, fa[buf][i]), __builtin_bit_cast(bf16x8, fb[buf][jn]), acc[i][jn], 0, 0, 0);
      } else {
        // (bit-cast the whole chunk first: a bit_cast of a single vector
        // element lvalue is miscompiled into a read of element 0)
#pragma unroll
        for (int e = 0; e < E; ++e)
#pragma unroll
          for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int jn = 0; jn < NB; ++jn) {
              const f32x4 a4 = __builtin_bit_cast(f32x4, fa[buf][i]);
              const f32x4 b4 = __builtin_bit_cast(f32x4, fb[buf][jn]);
              acc[i][jn] = __builtin_amdgcn_mfma_f32_32x32x2f32(a4[e], b4[e], acc[i][jn], 0, 0, 0);
            }
      }
    };

    const int steps = chunk_steps(item.k_len, S::KS);
    if constexpr (S::kAhead) {
      // A wave is alone on its SIMD here, or a quarter's with one other: a quarter's K step took
      // 0.35 us of which the matrix instructions are 0.11, the rest being waits for fragments read
      // just before their use and the checks of the edge step.  So the fragments of step
      // s + 1 are read, step s + 2 is written to LDS and step s + 4 loaded while step s is
      // multiplied, and steps that are not near the last one check nothing.  Stage s % 2 is
      // free then: step s's fragments were read before the barrier that ended step s - 1.
      // Quarters, execute alone, us, before / after, layouts NN, NT, TN, operands in L2: 16 items of 128
      // 5.3 / 5.0, 5.6 / 5.0, 4.7 / 4.6, of 512 9.5 / 8.2, 10.6 / 8.6, 8.2 / 6.9, of 2048
      // 25.8 / 19.9, 30.5 / 22.2, 22.1 / 16.2; 32 items (two workgroups on a CU) of 256 8.0 / 7.5,
      // 8.7 / 7.9, 6.9 / 6.7, of 1000 17.5 / 16.6, 21.2 / 19.0, 15.8 / 14.5.  (Four register sets
      // instead of two: equal.)
      u32x4 ga[2][S::kSub], gb[2][S::kSub];
      auto read_sub = [&](auto stage_tag, auto ks_tag) {
        constexpr int P = decltype(stage_tag)::value, KSUB = decltype(ks_tag)::value;
        const unsigned char* stage = smem + P * S::kStage;
        ga[P][KSUB] = read_frag(stage, a_addr, std::bool_constant<A_K>{}, int_c<TM>{}, ks_tag, 0);
        gb[P][KSUB] = read_frag(stage, b_addr, std::bool_constant<B_K>{}, int_c<TN>{}, ks_tag, 0);
      };
      // (barriers to the scheduler: left alone it moves the reads down to their use)
      auto mma_sub = [&](int p, int x) {
        fa[0][0] = ga[p][x];
        fb[0][0] = gb[p][x];
        mma(0);
        __builtin_amdgcn_sched_barrier(0);
      };
      fetch(int_c<0>{}, 0);
      fetch(int_c<1>{}, 1);
      if (b != blockIdx.x) CLEAVE_LDS_BARRIER();   // every wave is past the previous item's last fragment reads
      commit(int_c<0>{}, int_c<0>{}, 0);
      fetch(int_c<0>{}, 2);
      CLEAVE_LDS_BARRIER();
      read_sub(int_c<0>{}, int_c<0>{});
      read_sub(int_c<0>{}, int_c<1>{});
      read_sub(int_c<0>{}, int_c<2>{});
      read_sub(int_c<0>{}, int_c<3>{});
      if (steps > 1) commit(int_c<1>{}, int_c<1>{}, 1);
      fetch(int_c<1>{}, 3);
      CLEAVE_LDS_BARRIER();
      auto k_step = [&](auto phase_tag, auto inner_tag, int s) {
        constexpr int P = decltype(phase_tag)::value, O = P ^ 1;
        constexpr bool INNER = decltype(inner_tag)::value;
        read_sub(int_c<O>{}, int_c<0>{});
        read_sub(int_c<O>{}, int_c<1>{});
        mma_sub(P, 0);
        read_sub(int_c<O>{}, int_c<2>{});
        read_sub(int_c<O>{}, int_c<3>{});
        mma_sub(P, 1);
        if constexpr (INNER) {
          ta.store(va[P], smem + P * S::kStage, t);
          tb.store(vb[P], smem + P * S::kStage + S::kATile, t);
          ta.load_inner(va[P]);
          tb.load_inner(vb[P]);
        } else if (s + 2 < steps) {
          commit(int_c<P>{}, int_c<P>{}, s + 2);
          fetch(int_c<P>{}, s + 4);
        }
        mma_sub(P, 2);
        mma_sub(P, 3);
        CLEAVE_LDS_BARRIER();
      };
      int s = 0;
      for (; s + 6 < steps; s += 2) {   // the turn's last load is of step s + 5, not of the last step (the edge step)
        k_step(int_c<0>{}, std::true_type{}, s);
        k_step(int_c<1>{}, std::true_type{}, s + 1);
      }
      while (s < steps) {
        k_step(int_c<0>{}, std::false_type{}, s);
        if (++s >= steps) break;
        k_step(int_c<1>{}, std::false_type{}, s);
        ++s;
      }
    } else {
      // Steps 0 .. SETS-1 into registers, step 0 on into LDS, step SETS behind it.
      fetch(int_c<0>{}, 0);
      if constexpr (SETS > 1) fetch(int_c<1>{}, 1);
      if (b != blockIdx.x) CLEAVE_LDS_BARRIER();   // every wave is past the previous item's last fragment reads
      commit(int_c<0>{}, int_c<0>{}, 0);
      fetch(int_c<0>{}, SETS);
      CLEAVE_LDS_BARRIER();
      read_frags(0, int_c<0>{}, 0);

      // Step s sits in LDS stage s % 2; register set s % SETS holds step s until
      // it is written to LDS at the end of step s - 1 (the stage's readers, step
      // s - 2's, are past the barrier between), and then takes step s + SETS.
      auto k_step = [&](auto phase_tag, int s) {
        constexpr int P = decltype(phase_tag)::value;
        constexpr int cur = P & 1, oth = cur ^ 1, next_set = (P + 1) % SETS;
        read_frags(cur, int_c<1>{}, 1);
        mma(0);
        read_frags(cur, int_c<2>{}, 0);
        mma(1);
        read_frags(cur, int_c<3>{}, 1);
        mma(0);
        if (s + 1 < steps) {
          commit(int_c<next_set>{}, int_c<oth>{}, s + 1);
          fetch(int_c<next_set>{}, s + 1 + SETS);
          CLEAVE_LDS_BARRIER();
          read_frags(oth, int_c<0>{}, 0);
        }
        mma(1);
      };
      for (int s = 0; s < steps;) {
        k_step(int_c<0>{}, s);
        if (++s >= steps) break;
        k_step(int_c<1>{}, s);
        if (++s >= steps) break;   // (not left to the loop's condition: the other form spills registers)
      }
    }

    const int row0 = wm * S::WTM + lh * 4;
    const int col0 = wn * S::WTN + l32;
    TileTarget target = tile_target(args, item);
    target.base += (m_off * target.ld + n_off) * (args.C && args.c_bf16 ? 2 : 4);
    if constexpr (S::BLK == 16) {
      store_block(acc[0][0], target, args.C && args.c_bf16, wm * S::WTM + 4 * (lane >> 4), col0, m_valid, n_valid);
    } else {
      store_tile<MB, NB>(acc, target, args.C && args.c_bf16, row0, col0, m_valid, n_valid,
                         m_valid == TM && n_valid == TN);
    }
  }
}

template <typename S, Storage A, Storage B>
hipError_t launch_one(const ExecuteArgs& args, int grid, hipStream_t stream) {
  hipLaunchKernelGGL((execute_kernel<S, A, B>), dim3(grid), dim3(S::NT), 2 * S::kStage, stream, args);
  return hipGetLastError();
}

template <typename S, Storage A, Storage B>
hipError_t configure_one() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(execute_kernel<S, A, B>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, 2 * S::kStage);
}

template <typename S>
hipError_t configure_layouts() {
  hipError_t e = configure_one<S, kByK, kByK>();
  if (e == hipSuccess) e = configure_one<S, kByK, kByRow>();
  if (e == hipSuccess) e = configure_one<S, kByRow, kByK>();
  if (e == hipSuccess) e = configure_one<S, kByRow, kByRow>();
  return e;
}

template <typename S>
hipError_t configure_elements() {
  hipError_t e = configure_one<S, kElements, kElements>();
  if (e == hipSuccess) e = configure_one<S, kElements, kByK>();
  if (e == hipSuccess) e = configure_one<S, kElements, kByRow>();
  if (e == hipSuccess) e = configure_one<S, kByK, kElements>();
  if (e == hipSuccess) e = configure_one<S, kByRow, kElements>();
  return e;
}

// Grid of a launch over work items of one class, and the workgroup tiles per item.
template <typename S>
int cut_items(ExecuteArgs* args, int tile_class, const GeneralLoads& how) {
  static_assert((kSmallTileRows % S::TM == 0 || S::TM == kLargeTileRows) && kLargeTileRows % S::TM == 0 &&
                (kSmallTileCols % S::TN == 0 || S::TN == kLargeTileCols) && kLargeTileCols % S::TN == 0,
                "a work item is cut into whole workgroup tiles");
  args->parts_m = parts_along(how.list.rows, tile_rows(tile_class), S::TM);
  args->parts_n = parts_along(how.list.cols, tile_cols(tile_class), S::TN);
  const int64_t blocks = (args->n_items + 7) / 8 * 8 * args->parts_m * args->parts_n;
  // (only for the two shapes that the figures beside general_workgroups are of)
  constexpr bool kTakesSecond = S::BLK == 32 && S::SETS == 2 && S::WPE == 4;
  const int64_t resident = static_cast<int64_t>(how.cus) * (S::WPE * 4 / (S::NT / 64));
  return general_workgroups(blocks, resident, kTakesSecond ? second_tiles_taken_up_to(resident, S::TM, how.list) : 0);
}

template <typename S>
hipError_t launch_layouts(ExecuteArgs args, int tile_class, const GeneralLoads& how, hipStream_t stream) {
  const int grid = cut_items<S>(&args, tile_class, how);
  const bool a_k = !args.transA;   // A stored M x K: K-contiguous
  const bool b_k = args.transB;    // B stored N x K: K-contiguous
  if (a_k && b_k) return launch_one<S, kByK, kByK>(args, grid, stream);
  if (a_k && !b_k) return launch_one<S, kByK, kByRow>(args, grid, stream);
  if (!a_k && b_k) return launch_one<S, kByRow, kByK>(args, grid, stream);
  return launch_one<S, kByRow, kByRow>(args, grid, stream);
}

// how.a_elements / how.b_elements: at least one of them.
template <typename S>
hipError_t launch_elements(ExecuteArgs args, int tile_class, const GeneralLoads& how, hipStream_t stream) {
  const int grid = cut_items<S>(&args, tile_class, how);
  if (how.a_elements && how.b_elements) return launch_one<S, kElements, kElements>(args, grid, stream);
  if (how.a_elements)
    return args.transB ? launch_one<S, kElements, kByK>(args, grid, stream)
                       : launch_one<S, kElements, kByRow>(args, grid, stream);
  return args.transA ? launch_one<S, kByRow, kElements>(args, grid, stream)
                     : launch_one<S, kByK, kElements>(args, grid, stream);
}

// Quarters of the 64 x 64 tile, a 16 x 16 block per wave, for launches of few fp32
// items (general_tile in api.cpp).
using Quarter = Shape<4, 32, 32, 2, 2, 2, 4>;
// Eight waves of 32 x 64: two on each SIMD where a launch leaves a CU one workgroup,
// four where it has two.  us, four waves of 64 x 64 / eight, layouts NN, NT, TN: bf16, 192
// items of 11 steps 17.3 / 15.2, 16.9 / 15.1, 17.7 / 15.5, 320 of 21 37.5 / 33.0, 36.2 /
// 33.6, 35.6 / 33.1, 1152 of 11 54.7 / 50.9, 54.8 / 53.6, 52.6 / 51.5, 768 of 3 18.9 / 18.3,
// 18.7 / 19.3, 18.6 / 18.3; fp32, 768 items of 32 steps 195 / 184, 187 / 185, 186 / 184,
// 4096^3 1012 / 967.
template <int EB>
using Wide = Shape<EB, 128, 128, 4, 2, 2, 4>;
// (which launches run it: four_waves in kernels.h)
template <int EB>
using Wide4 = Shape<EB, 128, 128, 2, 2, 2, 2>;
using Large = Shape<2, kLargeTileRows, kLargeTileCols, 2, 4, 1, 2>;
template <int EB>
using Narrow = Shape<EB, 64, 64, 2, 2, 2, 4>;
// Read ahead as the quarters do, 180 registers instead of 126, for launches of at most one
// 64 x 64 workgroup per CU whose longest chunk has eight steps or more (runs_lone).  us, Narrow / Lone,
// layouts NN, NT, TN: fp32, 64 items, 4 steps 6.8 / 6.9, 6.4 / 6.6, 6.8 / 6.9, 8 steps 9.4 / 9.3,
// 9.1 / 8.9, 9.5 / 9.2, 24 steps 20.1 / 17.5, 19.9 / 17.5, 20.3 / 17.6, 64 steps 47.2 / 38.9,
// 47.4 / 38.9, 47.9 / 39.1; bf16, rows not 16-byte aligned, operands from HBM, 16 items, 4 steps
// 5.3 / 5.5, 5.3 / 5.3, 5.5 / 5.7, 8 steps 8.0 / 7.7, 7.2 / 7.0, 8.3 / 7.8, 40 steps 22.3 / 17.5,
// 22.5 / 17.4, 22.8 / 17.7, 64 items of 40 22.9 / 18.1, 22.9 / 18.3, 23.4 / 18.3.  With two
// workgroups on a CU steps without edge checks were 1-8 % slower (128 and 384 items of 24).
template <int EB>
using Lone = Shape<EB, 64, 64, 2, 2, 2, 2>;
template <int EB>
using ByElement = Shape<EB, 64, 64, 2, 2, 1, 4>;

template <int EB>
hipError_t configure_type() {
  hipError_t e = configure_layouts<Wide<EB>>();
  if (e == hipSuccess) e = configure_layouts<Narrow<EB>>();
  if (e == hipSuccess) e = configure_layouts<Lone<EB>>();
  if (e == hipSuccess) e = configure_elements<ByElement<EB>>();
  if (EB == 4 && e == hipSuccess) e = configure_layouts<Quarter>();
  if (EB == 2 && e == hipSuccess) e = configure_one<Large, kByK, kByK>();
  if (e == hipSuccess) e = configure_one<Wide4<EB>, kByK, kByK>();
  if (e == hipSuccess) e = configure_one<Wide4<EB>, kByRow, kByRow>();
  if (EB == 4 && e == hipSuccess) e = configure_one<Wide4<4>, kByRow, kByK>();
  return e;
}

template <int EB>
hipError_t launch_type(const ExecuteArgs& args, int tile_class, const GeneralLoads& how, hipStream_t stream) {
  if (how.a_elements || how.b_elements)
    return launch_elements<ByElement<EB>>(args, tile_class, how, stream);
  if (EB == 2 && how.tile == kTileHuge) {   // large items, both operands K-contiguous
    ExecuteArgs whole = args;
    const int grid = cut_items<Large>(&whole, tile_class, how);
    return launch_one<Large, kByK, kByK>(whole, grid, stream);
  }
  if (how.tile == kTileWide4) {   // NT, TN and, fp32 only, TT
    ExecuteArgs cut = args;
    const int grid = cut_items<Wide4<EB>>(&cut, tile_class, how);
    if (!args.transA) return launch_one<Wide4<EB>, kByK, kByK>(cut, grid, stream);
    if (EB == 4 && args.transB) return launch_one<Wide4<4>, kByRow, kByK>(cut, grid, stream);
    return launch_one<Wide4<EB>, kByRow, kByRow>(cut, grid, stream);
  }
  if (EB == 4 && how.tile == kTileQuarter) return launch_layouts<Quarter>(args, tile_class, how, stream);
  if (how.tile == kTileLone) return launch_layouts<Lone<EB>>(args, tile_class, how, stream);
  return how.tile == kTileNarrow ? launch_layouts<Narrow<EB>>(args, tile_class, how, stream)
                                 : launch_layouts<Wide<EB>>(args, tile_class, how, stream);
}

}  // namespace

hipError_t configure_execute_kernels() {
  const hipError_t e = configure_type<2>();
  return e != hipSuccess ? e : configure_type<4>();
}

hipError_t launch_execute(const ExecuteArgs& args, int dtype, int tile_class, const GeneralLoads& how,
                          hipStream_t stream) {
  return dtype == CLEAVE_BF16 ? launch_type<2>(args, tile_class, how, stream)
                              : launch_type<4>(args, tile_class, how, stream);
}

}  // namespace cleave
