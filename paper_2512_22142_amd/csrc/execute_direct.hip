// bf16 sub-GEMM executor, fast path: operand tiles go from global memory
// straight into LDS (no register staging), through a ring of stages.
//
// Same contract as the general executor (paper Sec. 4.1: a task multiplies its
// rows of A with its columns of B over its chunk of the inner dimension and
// stores an fp32 partial block); used when every 16 bytes it fetches belong to one
// chunk and one tile and are aligned.
//
// The kernel is a template over its shape (workgroup tile, wave grid, ring
// depth); a wave owns a grid of 16 x 16 blocks, computed by MFMA 16x16x32 with
// fp32 accumulators in registers.  Its four shapes are at the end of the file,
// each for the four layouts of the operands, with and without chunks that end
// within a step.  What bounds full launches is the board's power, and this
// instruction does the same arithmetic for less of it than the 32 x 32 one (half
// of the accumulator traffic per product): products from registers, random
// operands, 2.05 against 1.82 PFLOP/s, the same bits.  Together with fewer
// instructions per K step: 4096 x 4096 x 4096 in 512 x 512 tiles, 4 splits 139 ->
// 131 us, 4096 x 4096 x 11008 320 -> 292 us, 16384 x 5120 x 13824 in 8 splits 2.06
// -> 1.95 ms.
//
// A wave-wide direct load writes 64 consecutive 16-byte LDS slots (lane l ->
// slot l), so the LDS layout is chosen through which global 16 bytes a lane
// fetches:
//   * K-contiguous operand (tile row r, CPR = 8 chunks of 8 k per step):
//       slot = r*CPR + (chunk ^ ((r>>1)&7));
//     16 consecutive rows at one chunk then cover 16 distinct bank groups (and
//     so do half of them at one chunk and half at its neighbour), so the
//     16-byte fragment reads are conflict free.
//   * operand stored with the tile-row index contiguous (read "transposed"):
//     the tile is kept as 64 k rows of R/8 chunks,
//       slot = k*(R/8) + (chunk ^ swizzle(k)),
//       swizzle = 4*(k & 3) ^ 2*((k >> 3) & 1),  for R = 64 4*((k >> 1) & 1) ^ 2*((k >> 3) & 1);
//     fragments are gathered with the LDS transpose read (ds_read_b64_tr_b16:
//     within 16 lanes, lane i supplies the address of 4 consecutive elements of
//     k row i/4 and receives column i of the 4 x 16 block), two reads per
//     fragment; the XOR spreads over the banks the eight k rows that 32 lanes
//     read.
//
// Stores: through a row-major image per wave in LDS behind the ring (store_rows).
//
// Order of accumulation per output element: ascending K steps, inside a step
// ascending k -- a function of the task record only (and the same for every
// shape, and for the general kernel's 32x32x16 instruction), hence bitwise
// reproducible on re-issue.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>
#include <utility>

#include "kernels.h"
#include "tile_store.h"
#include "plan_internal.h"

namespace cleave {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_void;
typedef __attribute__((address_space(3))) s16x4* lds_s16x4;

// Shape of the kernel: workgroup tile TM x TN computed by WM x WN waves, BK
// elements of K per step, STAGES ring stages.  ONE_ITEM: the launch has a
// workgroup for every item (or part of one), which none follows.
template <int TM_, int TN_, int WM_, int WN_, int BK_, int STAGES_, bool ONE_ITEM_>
struct Shape {
  static constexpr int TM = TM_, TN = TN_, WM = WM_, WN = WN_, BK = BK_, STAGES = STAGES_;
  static constexpr bool ONE_ITEM = ONE_ITEM_;
  static constexpr int NW = WM * WN;            // waves
  static constexpr int NT = NW * 64;            // threads
  static constexpr int WTM = TM / WM, WTN = TN / WN;   // wave tile
  static constexpr int MB = WTM / 16, NB = WTN / 16;   // 16 x 16 MFMA blocks per wave tile
  static constexpr int CPR = BK / 8;            // 16-byte chunks per K-contiguous row and step
  static constexpr int kSub = BK / 32;          // MFMA sub-steps per step
  static constexpr int kATile = TM * BK * 2;    // bytes
  static constexpr int kBTile = TN * BK * 2;
  static constexpr int kStage = kATile + kBTile;
  static constexpr int kLoadsA = kATile / 1024 / NW;   // wave-wide loads per wave and step
  static constexpr int kLoadsB = kBTile / 1024 / NW;
  static constexpr int kLoadsPerStep = kLoadsA + kLoadsB;
  // A tile smaller than the small class's: a workgroup computes one of the
  // PARTS_M x PARTS_N parts of a work item, and only that.
  static constexpr int PARTS_M = TM < kSmallTileRows ? kSmallTileRows / TM : 1;
  static constexpr int PARTS_N = TN < kSmallTileCols ? kSmallTileCols / TN : 1;
  static constexpr int PARTS = PARTS_M * PARTS_N;
  static_assert(kATile % (1024 * NW) == 0 && kBTile % (1024 * NW) == 0, "tile / wave count");
  static_assert(PARTS == 1 || ONE_ITEM, "a workgroup computes one part of an item");
  static_assert(BK == 64, "two sub-steps, full lines");
  static_assert(WTM % 32 == 0 && WTN % 32 == 0 && STAGES >= 2 && (STAGES & (STAGES - 1)) == 0, "shape");
};

// Waits until at most `n` vector-memory operations of this wave are still in
// flight (loads return in order, so the n youngest) and all of its LDS reads
// have returned, then joins the workgroup barrier.  The wait and the barrier
// sit in one asm statement with a memory clobber: the compiler can neither
// move LDS accesses or direct loads across it nor separate the two, and
// (unlike __syncthreads) it adds no wait for the younger loads.
#define CLEAVE_WAIT_BARRIER(n) \
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(n) : "memory")

template <int V>
using int_c = std::integral_constant<int, V>;

// XOR applied to the chunk index of a K-contiguous row so that 16 consecutive
// rows at one logical chunk fall into 16 different 16-byte bank groups.
__device__ __forceinline__ int row_swizzle(int r) { return (r >> 1) & 7; }

// XOR applied to the chunk index of k row `k` of a tile kept as k rows of CH
// chunks: spreads over the banks the eight k rows that half a wave's transpose
// read touches (four neighbours, and four of the next eight).
template <int CH>
__device__ __forceinline__ int k_swizzle(int k) {
  return (CH == 8 ? 4 * ((k >> 1) & 1) : 4 * (k & 3)) ^ (2 * ((k >> 3) & 1));
}

__device__ __align__(16) const unsigned char g_zeros[16] = {};

template <typename S, bool KCONTIG, int R>
struct DirectTile {
  static constexpr int kLoads = R * S::BK * 2 / 1024 / S::NW;
  static constexpr int CH = R / 8;     // chunks per k row (transposed layout)
  uint32_t goff[kLoads];

  __device__ __forceinline__ void init(int64_t row_stride, int64_t k_stride, int r_valid, int wave,
                                       int lane) {
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const int slot = (wave * kLoads + i) * 64 + lane;
      if constexpr (KCONTIG) {
        const int r = slot / S::CPR;
        const int c = (slot % S::CPR) ^ row_swizzle(r);
        goff[i] = static_cast<uint32_t>((min(r, r_valid - 1) * row_stride + c * 8) * 2) + (kLoads - 1 - i) * 1024;
      } else {
        const int k = slot / CH;
        const int c = (slot % CH) ^ k_swizzle<CH>(k);
        goff[i] = static_cast<uint32_t>((k * k_stride + min(c * 8, r_valid - 8)) * 2) + (kLoads - 1 - i) * 1024;
      }
    }
  }

  // gbase: the tile's first row at this step's first k (wave-uniform);
  // lds_tile: LDS byte address of the tile.  The loads are issued through inline
  // asm (scalar base + per-lane 32-bit offset, LDS base in M0) for two
  // reasons: no VALU address arithmetic in the K loop, and the compiler does
  // not see an LDS-writing vector-memory operation -- it would otherwise wait
  // for every load in flight before each LDS transpose read.  The statement
  // has no register outputs, so nothing the compiler may spill or reuse is
  // written asynchronously; completion is awaited with CLEAVE_WAIT_BARRIER.
  // M0 is on the clobber list so that the compiler keeps no value of its own
  // in M0 across the statement (it is a reserved register, hence the
  // diagnostic silenced here; nothing needs it preserved).  A wave's loads of a
  // tile fill neighbouring kilobytes of LDS under one M0: the instruction's
  // offset counts for both addresses, which the lane offsets and the base make
  // up for.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
  // L loads from the FIRST-th.
  template <int FIRST, int L>
  __device__ __forceinline__ void issue(const unsigned char* gbase, uint32_t lds_tile, int wave) const {
    const uint32_t lds = lds_tile + wave * (kLoads * 1024);
    const unsigned char* base = gbase - (kLoads - 1) * 1024;
    if constexpr (L == 4) {
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
                   "global_load_lds_dwordx4 %1, %5\n\tglobal_load_lds_dwordx4 %2, %5 offset:1024\n\t"
                   "global_load_lds_dwordx4 %3, %5 offset:2048\n\tglobal_load_lds_dwordx4 %4, %5 offset:3072"
                   :
                   : "s"(lds), "v"(goff[0]), "v"(goff[1]), "v"(goff[2]), "v"(goff[3]), "s"(base)
                   : "memory", "m0");
    } else if constexpr (L == 2) {
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
                   "global_load_lds_dwordx4 %1, %3 offset:%4\n\tglobal_load_lds_dwordx4 %2, %3 offset:%5"
                   :
                   : "s"(lds), "v"(goff[FIRST]), "v"(goff[FIRST + 1]), "s"(base), "n"(1024 * FIRST), "n"(1024 * FIRST + 1024)
                   : "memory", "m0");
    } else {
      static_assert(L == 1, "the statements above");
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%3"
                   :
                   : "s"(lds), "v"(goff[FIRST]), "s"(base), "n"(1024 * FIRST)
                   : "memory", "m0");
    }
  }

  // The same for a chunk's last step of which only k_valid of the BK elements
  // exist: lanes whose 16 bytes lie behind them fetch zeros, which add nothing.
  __device__ __forceinline__ void issue_tail(const unsigned char* gbase, uint32_t lds_tile, int wave, int lane_id,
                                             int k_valid) const {
    int lane = lane_id;
    asm volatile("" : "+v"(lane));   // computed here, not kept in registers through the K loop
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
      const int slot = (wave * kLoads + i) * 64 + lane;
      int k;   // the lane's first
      if constexpr (KCONTIG) k = ((slot % S::CPR) ^ row_swizzle(slot / S::CPR)) * 8;
      else k = slot / CH;
      const unsigned char* p = k < k_valid ? gbase + (goff[i] - (kLoads - 1 - i) * 1024) : g_zeros;
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                   :
                   : "s"(lds_tile + (wave * kLoads + i) * 1024), "v"(p)
                   : "memory", "m0");
    }
  }
#pragma clang diagnostic pop
};

// Order of a run of M MFMAs and READS LDS reads, as a hint to the scheduler: the
// reads spread evenly behind all but the last eighth of the MFMAs.
template <int M, int READS, int... I>
__device__ __forceinline__ void spread_reads_at(std::integer_sequence<int, I...>) {
  constexpr int kSlots = M > 4 ? M - M / 8 : M > 1 ? M - 1 : 1;
  constexpr auto done = [](int m) { return m >= kSlots ? READS : (m * READS + kSlots - 1) / kSlots; };
  ((__builtin_amdgcn_sched_group_barrier(0x008, 1, 0),
    __builtin_amdgcn_sched_group_barrier(0x100, done(I + 1) - done(I), 0)), ...);
}
template <int M, int READS>
__device__ __forceinline__ void spread_reads() {
  spread_reads_at<M, READS>(std::make_integer_sequence<int, M>{});
}

// TAILS: some chunk of the launch ends within a K step (the code for that costs
// scalar registers: an instantiation of its own).
template <typename S, bool A_K, bool B_K, bool TAILS>
__global__ __launch_bounds__(S::NT, 512 / S::NT) void execute_direct_kernel(ExecuteArgs args) {
  constexpr int TM = S::TM, TN = S::TN, MB = S::MB, NB = S::NB, CPR = S::CPR, kSub = S::kSub;
  constexpr int kStage = S::kStage, kATile = S::kATile, STAGES = S::STAGES, LPS = S::kLoadsPerStep;
  constexpr int kRowBytes = CPR * 16;        // K-contiguous tile row
  constexpr int CHA = TM / 8, CHB = TN / 8;  // chunks per k row, transposed tiles

  extern __shared__ __align__(16) unsigned char smem[];

  const int t = threadIdx.x;
  const int lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = wave / S::WN;
  const int wn = wave % S::WN;
  const int l16 = lane & 15;
  const int lq = lane >> 4;           // which 8 of a sub-step's 32 k

  // Lane-constant fragment addresses (byte offsets inside a stage).
  // K-contiguous: one per sub-step; blocks are 16 rows apart.  Transposed: one
  // per block (the XOR touches the block bits); sub-step and half select the k
  // rows through a constant offset.
  const uint32_t smem_off = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_void)smem));
  const int kq = l16 >> 2;            // k row (mod 4) this lane addresses in a transpose read
  const int cq = l16 & 3;             // which 4 of the 16 columns
  uint32_t a_addr[A_K ? kSub : MB];
  uint32_t b_addr[B_K ? kSub : NB];
  if constexpr (A_K) {
#pragma unroll
    for (int ks = 0; ks < kSub; ++ks)
      a_addr[ks] = (wm * S::WTM + l16) * kRowBytes + (((4 * ks + lq) ^ row_swizzle(l16)) * 16);
  } else {
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      const int c = wm * (S::WTM / 8) + i * 2 + (cq >> 1);
      a_addr[i] = ((8 * lq + kq) * CHA + (c ^ k_swizzle<CHA>(8 * lq + kq))) * 16 + (cq & 1) * 8;
    }
  }
  if constexpr (B_K) {
#pragma unroll
    for (int ks = 0; ks < kSub; ++ks)
      b_addr[ks] = kATile + (wn * S::WTN + l16) * kRowBytes + (((4 * ks + lq) ^ row_swizzle(l16)) * 16);
  } else {
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int c = wn * (S::WTN / 8) + j * 2 + (cq >> 1);
      b_addr[j] = kATile + ((8 * lq + kq) * CHB + (c ^ k_swizzle<CHB>(8 * lq + kq))) * 16 + (cq & 1) * 8;
    }
  }

  // Element strides of the stored operands along (tile row, K).
  const int64_t a_rs = args.transA ? 1 : args.lda;
  const int64_t a_ks = args.transA ? args.lda : 1;
  const int64_t b_rs = args.transB ? args.ldb : 1;
  const int64_t b_ks = args.transB ? 1 : args.ldb;

  // Everything a work item needs, wave-uniform (scalar registers).
  struct ItemCtx {
    const unsigned char* a_ptr;   // first row of the A tile at the first k that has not been fetched yet
    const unsigned char* b_ptr;
    TileTarget out;               // where this sub-tile's accumulators go
    int steps, m_valid, n_valid;
    int tail;                     // elements of the last step if it is not a whole one, else 0
  };
  auto load_item = [&](int64_t idx) -> WorkItem {
    if constexpr (S::PARTS == 1) {
      return load_work_item(args.items, idx);
    } else {
      // workgroups are dealt round-robin over the XCDs and list position i belongs to
      // XCD i % 8: the parts of an item follow each other on the item's XCD
      const uint32_t part = static_cast<uint32_t>(idx >> 3) % S::PARTS;
      const int64_t it = (idx >> 3) / S::PARTS * 8 + (idx & 7);
      WorkItem w = load_work_item(args.items, it < args.n_items ? it : 0);
      const uint32_t mo = part / S::PARTS_N * TM, no = part % S::PARTS_N * TN;
      const bool empty = it >= args.n_items || mo >= w.m_valid || no >= w.n_valid;
      w.m_valid = empty ? 0 : min(w.m_valid - mo, static_cast<uint32_t>(TM));
      w.n_valid = empty ? 0 : min(w.n_valid - no, static_cast<uint32_t>(TN));
      w.m_base += mo;
      w.n_base += no;
      w.out_off += static_cast<uint64_t>(mo) * w.out_ld + no;
      return w;
    }
  };
  auto make_ctx = [&](const WorkItem& w) -> ItemCtx {
    ItemCtx c;
    c.m_valid = static_cast<int>(w.m_valid);
    c.n_valid = static_cast<int>(w.n_valid);
    c.steps = chunk_steps(w.k_len, S::BK);
    c.tail = static_cast<int>(w.k_len % S::BK);
    c.a_ptr = static_cast<const unsigned char*>(args.A) +
              (member_offset(args.a_at, args.batch, w.gemm_id) +
               static_cast<int64_t>(w.m_base) * a_rs + static_cast<int64_t>(w.k0) * a_ks) * 2;
    c.b_ptr = static_cast<const unsigned char*>(args.B) +
              (member_offset(args.b_at, args.batch, w.gemm_id) +
               static_cast<int64_t>(w.n_base) * b_rs + static_cast<int64_t>(w.k0) * b_ks) * 2;
    c.out = tile_target(args, w);
    return c;
  };
  const int64_t a_step = a_ks * S::BK * 2;    // bytes per K step
  const int64_t b_step = b_ks * S::BK * 2;

  DirectTile<S, A_K, TM> ta;
  DirectTile<S, B_K, TN> tb;
  // Fetches the item's next step into ring stage st: A's part and B's, each at
  // once or in two halves.
  constexpr int_c<0> whole{};
  constexpr int_c<1> first_half{};
  constexpr int_c<2> second_half{};
  auto issue_a = [&](ItemCtx& c, int st, auto what) {
    constexpr int W = decltype(what)::value, L = S::kLoadsA / (W ? 2 : 1);
    ta.template issue<W == 2 ? L : 0, L>(c.a_ptr, smem_off + st * kStage, wave);
    if (W != 1) c.a_ptr += a_step;
  };
  auto issue_b = [&](ItemCtx& c, int st, auto what) {
    constexpr int W = decltype(what)::value, L = S::kLoadsB / (W ? 2 : 1);
    tb.template issue<W == 2 ? L : 0, L>(c.b_ptr, smem_off + st * kStage + kATile, wave);
    if (W != 1) c.b_ptr += b_step;
  };
  auto issue = [&](ItemCtx& c, int s, int st) {   // s: that step, which may be the chunk's last
    if (TAILS && c.tail != 0 && s == c.steps - 1) {
      ta.issue_tail(c.a_ptr, smem_off + st * kStage, wave, lane, c.tail);
      tb.issue_tail(c.b_ptr, smem_off + st * kStage + kATile, wave, lane, c.tail);
      return;
    }
    issue_a(c, st, whole);
    issue_b(c, st, whole);
  };
  // Start of a work item: lane offsets for its (possibly clipped) tile, then
  // the first STAGES steps into the ring.
  auto fill_ring = [&](ItemCtx& c) {
    ta.init(a_rs, a_ks, c.m_valid, wave, lane);
    tb.init(b_rs, b_ks, c.n_valid, wave, lane);
#pragma unroll
    for (int st = 0; st < STAGES; ++st)
      if (st < c.steps) issue(c, st, st);
  };

  // A workgroup walks its work items -- every grid-th one, or a run of its own
  // when the launch comes with a balanced schedule.  The ring runs on across
  // items: when the current item and the next one are both full sub-tiles of at
  // least a ring's worth of steps, the next item's first steps are fetched into
  // the stages that this item's last steps free, exactly as this item's own
  // later steps would be, so the next K loop starts without a ring fill and
  // without waiting for this item's stores.  Otherwise (clipped sub-tiles need
  // other lane offsets) the ring is filled from empty after the item's last
  // step, ahead of its stores.
  //
  // Store instructions per lane of a full sub-tile.
  const bool bf16_out = args.C && args.c_bf16;
  const int tile_stores = bf16_out ? MB * NB / 2 : MB * NB;
  unsigned char* const image = smem + STAGES * kStage + wave * kBlockImageBytes;

  // This workgroup's items: first, first + stride, ... below it_end.
  int64_t it_first = blockIdx.x, it_end = args.n_items, stride = gridDim.x;
  if (!S::ONE_ITEM && args.wg_ranges) {
    it_first = args.wg_ranges[blockIdx.x];
    it_end = args.wg_ranges[blockIdx.x + 1];
    stride = 1;
  }
  if constexpr (S::ONE_ITEM) it_end = it_first + 1;
  if (it_first >= it_end) return;
  ItemCtx c = make_ctx(load_item(it_first));
  if (S::PARTS > 1 && c.m_valid == 0) return;
  fill_ring(c);
  int64_t it_next = it_first + stride;
  // Item records are read two items ahead (scalar loads through the constant
  // address space): the read for the item after next is issued right behind
  // the current item's first barrier, a whole K step before the next wait
  // that covers it.  `last_item` stands in for records past the end.
  const int64_t last_item = it_end - 1;
  ItemCtx nx = S::ONE_ITEM ? c : make_ctx(load_item(it_next < it_end ? it_next : last_item));
  WorkItem after_next;
  // How the current item's first steps got into the ring.
  //   kFilled:             ring filled from empty; what has been issued since, if
  //     anything, is not counted.
  //   kFilledBehindStores: ring filled from empty, then exactly the tile_stores
  //     stores of the previous item.
  //   kPrefetched:         fetched during the previous item's last steps, then its
  //     tile_stores stores; step 0 was waited for at that item's last barrier
  //     (its first fragments are already in registers).
  // The counter of outstanding operations retires in issue order, so a step has
  // landed once at most the operations issued behind it are outstanding: the
  // later steps in the ring and, for the steps fetched ahead of them, the
  // stores, none of which has to complete for that.
  enum Entry : int { kFilled = 0, kFilledBehindStores = 1, kPrefetched = 2 };
  int entry = kFilled;
  int phase = 0;   // ring stage that holds the current item's step 0
  // Barrier once at most `steps_behind` steps' loads and `stores` stores are
  // outstanding.  (The counts are multiples of four; the counter holds 63.)
  static_assert(LPS % 4 == 0 && (STAGES - 1) * LPS + MB * NB <= 40, "the wait counts below");
  auto wait_behind = [&](int steps_behind, int stores) {
    switch ((steps_behind * LPS + stores) >> 2) {
      case 0: CLEAVE_WAIT_BARRIER(0); break;
      case 1: CLEAVE_WAIT_BARRIER(4); break;
      case 2: CLEAVE_WAIT_BARRIER(8); break;
      case 3: CLEAVE_WAIT_BARRIER(12); break;
      case 4: CLEAVE_WAIT_BARRIER(16); break;
      case 5: CLEAVE_WAIT_BARRIER(20); break;
      case 6: CLEAVE_WAIT_BARRIER(24); break;
      case 7: CLEAVE_WAIT_BARRIER(28); break;
      case 8: CLEAVE_WAIT_BARRIER(32); break;
      case 9: CLEAVE_WAIT_BARRIER(36); break;
      default: CLEAVE_WAIT_BARRIER(40); break;
    }
  };

  // A wave holds one sub-step's fragments, in halves of A's and B's that are
  // replaced as soon as they are done with; small wave tiles hold two sub-steps'.
  // (Two sub-steps' of the large tile spill; of 64 x 64 they are read in bursts:
  // 216 items of 64 steps 36.7 us, 34.6 in halves.)
  constexpr bool kQuarters = MB * NB >= 16;
  // The refill's loads leave in two groups, or in four where a wave may be alone on
  // its SIMD and its MFMAs stand behind the queue of the address unit (288 items
  // of 64 steps: 51.8 us all at once, 49.9 in two groups, 48.5 in four; large
  // tiles 2.02 / 1.95 / 2.00 ms for 16384 x 5120 x 13824).
  constexpr bool kPairs = S::NW == 8;
  constexpr int MH = MB / 2, NH = NB / 2;
  f32x4 acc[MB][NB];
  u32x4 fa[kQuarters ? 1 : 2][MB], fb[kQuarters ? 1 : 2][NB];

  // Fragment reads are ordinary (compiler-visible) LDS loads: the compiler
  // tracks their completion, and every address is a lane-constant register
  // plus a compile-time offset (stage, block, sub-step).
  auto tr_read = [&](const unsigned char* p) -> u32x2 {
    return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)p));
  };
  // Fragments I0 .. I0 + N - 1 of A (of B) of sub-step KS of the ring stage at
  // byte offset `stage`.
  auto read_a = [&](uint32_t stage, auto ks_tag, auto i0_tag, auto n_tag) {
    constexpr int KS = decltype(ks_tag)::value, I0 = decltype(i0_tag)::value;
    constexpr int SET = kQuarters ? 0 : KS;
#pragma unroll
    for (int i = I0; i < I0 + decltype(n_tag)::value; ++i) {
      if constexpr (A_K) {
        fa[SET][i] = *reinterpret_cast<const u32x4*>(smem + (a_addr[KS] + stage) + i * 16 * kRowBytes);
      } else {
        const unsigned char* p = smem + (a_addr[i] + stage) + KS * (32 * CHA * 16);
        const u32x2 lo = tr_read(p);
        const u32x2 hi = tr_read(p + 4 * CHA * 16);
        fa[SET][i] = u32x4{lo[0], lo[1], hi[0], hi[1]};
      }
    }
  };
  auto read_b = [&](uint32_t stage, auto ks_tag, auto j0_tag, auto n_tag) {
    constexpr int KS = decltype(ks_tag)::value, J0 = decltype(j0_tag)::value;
    constexpr int SET = kQuarters ? 0 : KS;
#pragma unroll
    for (int j = J0; j < J0 + decltype(n_tag)::value; ++j) {
      if constexpr (B_K) {
        fb[SET][j] = *reinterpret_cast<const u32x4*>(smem + (b_addr[KS] + stage) + j * 16 * kRowBytes);
      } else {
        const unsigned char* p = smem + (b_addr[j] + stage) + KS * (32 * CHB * 16);
        const u32x2 lo = tr_read(p);
        const u32x2 hi = tr_read(p + 4 * CHB * 16);
        fb[SET][j] = u32x4{lo[0], lo[1], hi[0], hi[1]};
      }
    }
  };
  // Rows I0 .. I0 + M - 1 times columns J0 .. J0 + N - 1 of sub-step KS.  B is the
  // first operand, so that a lane ends up with four neighbouring columns of a
  // row.  Neighbouring products share a fragment (the columns are walked to and
  // fro).  `fresh`: the first product of a work item starts from zero (a constant
  // operand of the instruction: no pass over the accumulators to clear them).
  auto mma = [&](auto ks_tag, auto i0_tag, auto m_tag, auto j0_tag, auto n_tag, auto fresh_tag) {
    constexpr int SET = kQuarters ? 0 : decltype(ks_tag)::value;
    constexpr int I0 = decltype(i0_tag)::value, J0 = decltype(j0_tag)::value, N = decltype(n_tag)::value;
    constexpr bool FRESH = decltype(fresh_tag)::value;
#pragma unroll
    for (int x = 0; x < decltype(m_tag)::value; ++x)
#pragma unroll
      for (int y = 0; y < N; ++y) {
        const int i = I0 + x, j = J0 + (i & 1 ? N - 1 - y : y);
        f32x4 sum = acc[i][j];
        if constexpr (FRESH) sum = f32x4{};
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            __builtin_bit_cast(bf16x8, fb[SET][j]), __builtin_bit_cast(bf16x8, fa[SET][i]), sum, 0, 0, 0);
      }
  };
  constexpr int kReadsA = (A_K ? 1 : 2) * MB, kReadsB = (B_K ? 1 : 2) * NB;

  // How a step hands its ring stage on.
  //   kRefilled: at least STAGES more whole steps follow it and only the ring's own loads are
  //     outstanding: the stage is refilled, no case distinctions.
  //   kRefilledLast (ONE_ITEM): the same, but the step it is refilled with is the chunk's last
  //     and no whole one.
  //   1 .. STAGES (ONE_ITEM): that many steps are left, this one among them, all in the ring.
  //   kAnyStep (several items per workgroup): whatever applies.
  constexpr int kAnyStep = 100, kRefilled = 101, kRefilledLast = 102;

  for (;;) {
    const int steps = c.steps;
    const bool has_next = !S::ONE_ITEM && it_next < it_end;
    const bool interior = c.m_valid == TM && c.n_valid == TN;
    // hand the ring over without draining it
    const bool cont = has_next && interior && nx.m_valid == TM && nx.n_valid == TN && steps >= STAGES && nx.steps >= STAGES;
    // stores between the steps fetched ahead of the item and its own
    const int stores_behind = entry == kFilled ? 0 : tile_stores;

    // The fragments that a step begins with.
    auto first_frags = [&](uint32_t stage) {
      if constexpr (kQuarters) {
        read_a(stage, int_c<0>{}, int_c<0>{}, int_c<MH>{});
        read_b(stage, int_c<0>{}, int_c<0>{}, int_c<NH>{});
      } else {   // in the order in which they are multiplied
        read_a(stage, int_c<0>{}, int_c<0>{}, int_c<1>{});
        read_b(stage, int_c<0>{}, int_c<0>{}, int_c<NB>{});
        read_a(stage, int_c<0>{}, int_c<1>{}, int_c<MB - 1>{});
      }
    };

    // Step 0 must have landed.  All earlier fragment reads of this workgroup
    // completed before the previous item's final barrier.
    if (entry != kPrefetched) {
      wait_behind(min(STAGES, steps) - 1, stores_behind);
      first_frags(0u);   // a ring filled from empty starts at stage 0
    }

    // One K step; step s sits in ring stage (s + phase) % STAGES.  While the
    // fragments at hand are multiplied, later ones are fetched.  The barrier
    // sits where this wave holds all that it still needs of step s and the step
    // after it has landed (loads return in order), so the stage is refilled
    // with the step STAGES further on -- this item's, or one of the next item's
    // first -- and the first fragments of the following step are fetched behind
    // it, while the rest of the step multiplies.
    auto k_step = [&](auto how_tag, auto first_tag, int s) {
      constexpr int HOW = decltype(how_tag)::value;
      constexpr bool MID = HOW == kRefilled;
      constexpr std::bool_constant<decltype(first_tag)::value> fresh{};   // the item's step 0
      constexpr std::false_type more{};
      const int st = (s + phase) & (STAGES - 1);
      const uint32_t cur = st * kStage;
      const uint32_t oth = ((st + 1) & (STAGES - 1)) * kStage;
      const bool last = s + 1 >= steps;
      const bool go_on = HOW == kAnyStep ? !last || cont : HOW != 1;   // a step follows in the ring
      auto hand_over = [&]() {
        if constexpr (MID) {
          CLEAVE_WAIT_BARRIER((STAGES - 2) * LPS);
          if constexpr (!kQuarters) {
            issue_a(c, st, whole);
            issue_b(c, st, whole);
          } else if constexpr (kPairs) {
            issue_a(c, st, whole);
          } else {
            issue_a(c, st, first_half);
          }
        } else if constexpr (HOW == kRefilledLast) {
          CLEAVE_WAIT_BARRIER((STAGES - 2) * LPS);
          ta.issue_tail(c.a_ptr, smem_off + st * kStage, wave, lane, c.tail);
          tb.issue_tail(c.b_ptr, smem_off + st * kStage + kATile, wave, lane, c.tail);
        } else if constexpr (HOW != kAnyStep) {
          if constexpr (HOW > 1) CLEAVE_WAIT_BARRIER((HOW - 2) * LPS);
        } else {
          if (!go_on) {
            // nothing to wait for, and no reason to wait for the previous item's stores either
            CLEAVE_WAIT_BARRIER(63);
          } else {
            wait_behind(cont ? STAGES - 2 : min(STAGES - 2, steps - 2 - s), s + 1 < STAGES ? stores_behind : 0);
          }
          if (s + STAGES < steps) {
            issue(c, s + STAGES, st);
          } else if (cont) {
            issue(nx, s + STAGES - steps, st);
          }
          if (s == 0) after_next = load_item(it_next + stride < it_end ? it_next + stride : last_item);
        }
      };
      constexpr int_c<0> k0{};
      constexpr int_c<1> k1{};
      if constexpr (kQuarters) {
        // Four quarters per sub-step: (first half of A, one half of B), the other
        // half of B, then the second half of A with B's halves the other way
        // round, so that each half of B changes once per sub-step.
        constexpr int_c<0> lo{};
        constexpr int_c<MH> a_hi{}, mh{};
        constexpr int_c<NH> b_hi{}, nh{};
        read_b(cur, k0, b_hi, nh);
        mma(k0, lo, mh, lo, nh, fresh);
        spread_reads<MH * NH, kReadsB / 2>();
        read_a(cur, k0, a_hi, mh);
        mma(k0, lo, mh, b_hi, nh, fresh);
        spread_reads<MH * NH, kReadsA / 2>();
        read_a(cur, k1, lo, mh);
        mma(k0, a_hi, mh, b_hi, nh, fresh);
        spread_reads<MH * NH, kReadsA / 2>();
        read_b(cur, k1, b_hi, nh);
        mma(k0, a_hi, mh, lo, nh, fresh);
        spread_reads<MH * NH, kReadsB / 2>();
        read_b(cur, k1, lo, nh);
        mma(k1, lo, mh, b_hi, nh, more);
        spread_reads<MH * NH, kReadsB / 2>();
        read_a(cur, k1, a_hi, mh);
        mma(k1, lo, mh, lo, nh, more);
        spread_reads<MH * NH, kReadsA / 2>();
        hand_over();
        // The refill's loads are spread over the rest of the step.
        if constexpr (kPairs) {
          if (go_on) read_a(oth, k0, lo, mh);
          mma(k1, a_hi, mh, lo, nh, more);
          spread_reads<MH * NH, kReadsA / 2>();
          if constexpr (MID) issue_b(c, st, whole);
          if (go_on) read_b(oth, k0, lo, nh);
          mma(k1, a_hi, mh, b_hi, nh, more);
          spread_reads<MH * NH, kReadsB / 2>();
        } else {
          constexpr int_c<MH / 2> mq{};
          constexpr int_c<MH + MH / 2> a_last{};
          constexpr int_c<NH / 2> nq{};
          if (go_on) read_a(oth, k0, lo, mq);
          mma(k1, a_hi, mq, lo, nh, more);
          spread_reads<MH * NH / 2, kReadsA / 4>();
          if constexpr (MID) issue_a(c, st, second_half);
          if (go_on) read_a(oth, k0, mq, mq);
          mma(k1, a_last, mq, lo, nh, more);
          spread_reads<MH * NH / 2, kReadsA / 4>();
          if constexpr (MID) issue_b(c, st, first_half);
          if (go_on) read_b(oth, k0, lo, nq);
          mma(k1, a_hi, mq, b_hi, nh, more);
          spread_reads<MH * NH / 2, kReadsB / 4>();
          if constexpr (MID) issue_b(c, st, second_half);
          if (go_on) read_b(oth, k0, nq, nq);
          mma(k1, a_last, mq, b_hi, nh, more);
          spread_reads<MH * NH / 2, kReadsB / 4>();
        }
      } else {
        constexpr int_c<MB> m{};
        constexpr int_c<NB> n{};
        read_a(cur, k1, k0, k1);
        read_b(cur, k1, k0, n);
        read_a(cur, k1, k1, int_c<MB - 1>{});
        mma(k0, k0, m, k0, n, fresh);
        spread_reads<MB * NB, kReadsA + kReadsB>();
        hand_over();
        if (go_on) first_frags(oth);
        mma(k1, k0, m, k0, n, more);
        spread_reads<MB * NB, kReadsA + kReadsB>();
      }
    };
    const int full = steps - (TAILS && c.tail != 0);
    if constexpr (S::ONE_ITEM) {
      // The ring drains once: a copy of the step for each number of steps left, whose waits
      // are constants.  What bounds a lone workgroup is the time of a step, and through the
      // general form, with its branches between the matrix instructions, each of the first three
      // and last four steps of a chunk took 0.1 us longer.  us, that form / this: parts, 16 items
      // of 6 steps 4.7 / 4.1, of 16 6.5 / 5.7, 64 items of 8 5.8 / 4.9, 128 items of 16 9.9 / 9.1,
      // deep, 192 items of 16 13.9 / 12.9, of 32 20.5 / 19.1.
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = f32x4{};
      int s = 0;
      for (; s + STAGES < full; ++s) k_step(int_c<kRefilled>{}, std::false_type{}, s);
      if (TAILS && s + STAGES < steps) k_step(int_c<kRefilledLast>{}, std::false_type{}, s++);
      const int left = steps - s;
      static_assert(STAGES == 4, "the copies below");
      if (left > 3) k_step(int_c<4>{}, std::false_type{}, s++);
      if (left > 2) k_step(int_c<3>{}, std::false_type{}, s++);
      if (left > 1) k_step(int_c<2>{}, std::false_type{}, s++);
      k_step(int_c<1>{}, std::false_type{}, s);
    } else {
      static_assert(STAGES == 2, "a step behind step 0 has only the ring's own loads outstanding");
      k_step(int_c<kAnyStep>{}, std::true_type{}, 0);
      int s = 1;
      for (; s + STAGES < full; ++s) k_step(int_c<kRefilled>{}, std::false_type{}, s);
      for (; s < steps; ++s) k_step(int_c<kAnyStep>{}, std::false_type{}, s);
    }

    // With items to follow, every wave is past the last step's barrier, hence past all of its
    // fragment reads of this item.  A lone item's last step has none: nothing refills the ring,
    // and the stores' image lies behind it and is the wave's own.
    const TileTarget target = c.out;
    const int m_valid = c.m_valid, n_valid = c.n_valid;
    // The ring is free unless it was handed over: the next item's ring fill is
    // issued before this item's stores so that its latency hides behind them.
    if (!cont && has_next) fill_ring(nx);
    // (only the large shape has both forms: the second one's code alone cost launches of few
    // K steps of the others 1-2 %)
    constexpr bool kStreams = S::NW == 8;
    const auto leave = [&](auto bf16_tag, auto interior_tag, auto stream_tag) {
      store_rows<decltype(bf16_tag)::value, decltype(interior_tag)::value, decltype(stream_tag)::value, MB, NB>(
          acc, target, image, wm * S::WTM, wn * S::WTN, lane, m_valid, n_valid);
    };
    constexpr std::true_type yes{};
    constexpr std::false_type no{};
    if (!bf16_out) {
      if (!interior) leave(no, no, no);
      else if (kStreams && target.stream) leave(no, yes, yes);
      else leave(no, yes, no);
    } else {
      if (!interior) leave(yes, no, no);
      else if (kStreams && target.stream) leave(yes, yes, yes);
      else leave(yes, yes, no);
    }
    entry = cont ? kPrefetched : interior ? kFilledBehindStores : kFilled;
    phase = cont ? (phase + steps) & (STAGES - 1) : 0;
    if (!has_next) break;
    c = nx;
    nx = make_ctx(after_next);
    it_next += stride;
  }
}

template <typename S, bool A_K, bool B_K, bool TAILS>
hipError_t launch_one(const ExecuteArgs& args, int grid, hipStream_t stream) {
  constexpr size_t lds = S::STAGES * S::kStage + S::NW * kBlockImageBytes;
  hipLaunchKernelGGL((execute_direct_kernel<S, A_K, B_K, TAILS>), dim3(grid), dim3(S::NT), lds, stream, args);
  return hipGetLastError();
}

template <typename S, bool A_K, bool B_K, bool TAILS>
hipError_t configure_one() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(execute_direct_kernel<S, A_K, B_K, TAILS>),
                             hipFuncAttributeMaxDynamicSharedMemorySize,
                             static_cast<int>(S::STAGES * S::kStage + S::NW * kBlockImageBytes));
}

template <typename S, bool TAILS>
hipError_t configure_layouts() {
  hipError_t e = configure_one<S, true, true, TAILS>();
  if (e == hipSuccess) e = configure_one<S, true, false, TAILS>();
  if (e == hipSuccess) e = configure_one<S, false, true, TAILS>();
  if (e == hipSuccess) e = configure_one<S, false, false, TAILS>();
  return e;
}
template <typename S>
hipError_t configure_shape() {
  const hipError_t e = configure_layouts<S, false>();
  return e == hipSuccess ? configure_layouts<S, true>() : e;
}

// All shapes fetch full 128-byte lines of K-contiguous operands (64 elements of
// K per step).
//   large class: 256 x 256 tile, 8 waves (2 x 4, each 128 x 64), two 64 KB
//     stages, one workgroup per CU;
//   small class: 128 x 128 tile, 4 waves (each 64 x 64), two 32 KB stages, two
//     workgroups per CU;
//   deep: a launch with at most one small item per CU leaves half of the LDS
//     unused and a lone workgroup waiting for its loads, one step ahead.  Four
//     stages, three steps ahead, one workgroup per CU: 192 items of 24 steps
//     24.7 -> 18.5 us, of 12 12.9 -> 10.8, of 2 7.5 -> 6.6 (inputs not in any
//     cache; the other lengths are beside direct_shape); full launches lose the
//     second workgroup (4096 items of 16 steps 187 / 221 us);
//   parts: a launch of few small items has one short-lived workgroup per CU, or
//     none, and what bounds it is the time one K step takes a lone workgroup:
//     0.40 us at 128 x 128, of which its matrix instructions are 0.21.  64 x 64
//     parts (4 waves of 32 x 32) spread an item over four CUs, read and fill a
//     third of the LDS per step, and four 16 KB stages keep three steps' loads
//     in flight: 0.17 us per step.  Execute, 128 x 128 items -> parts: 32 items
//     of 6 steps 6.8 -> 4.1 us, 64 of 48 30 -> 13.2, 96 of 48 31 -> 19.9, 128 of
//     48 32 -> 22.8 us.  Full launches do better with the larger tile (4096
//     items of 16 steps 164 / 237 us).
using LargeShape = Shape<kLargeTileRows, kLargeTileCols, 2, 4, 64, 2, false>;
using SmallShape = Shape<kSmallTileRows, kSmallTileCols, 2, 2, 64, 2, false>;
using DeepShape = Shape<kSmallTileRows, kSmallTileCols, 2, 2, 64, 4, true>;
using PartsShape = Shape<64, 64, 2, 2, 64, 4, true>;
static_assert(kDirectKStep == LargeShape::BK && kDirectKStep == SmallShape::BK &&
              kDirectKStep == DeepShape::BK && kDirectKStep == PartsShape::BK, "the host's unit of cost");

template <typename S, bool TAILS>
hipError_t launch_layouts(const ExecuteArgs& args, int grid, hipStream_t stream) {
  const bool a_k = !args.transA;   // A stored M x K: K-contiguous
  const bool b_k = args.transB;    // B stored N x K: K-contiguous
  if (a_k && b_k) return launch_one<S, true, true, TAILS>(args, grid, stream);
  if (a_k && !b_k) return launch_one<S, true, false, TAILS>(args, grid, stream);
  if (!a_k && b_k) return launch_one<S, false, true, TAILS>(args, grid, stream);
  return launch_one<S, false, false, TAILS>(args, grid, stream);
}
template <typename S>
hipError_t launch_shape(const ExecuteArgs& args, bool tails, int grid, hipStream_t stream) {
  return tails ? launch_layouts<S, true>(args, grid, stream) : launch_layouts<S, false>(args, grid, stream);
}

}  // namespace


hipError_t configure_execute_direct_kernels() {
  hipError_t e = configure_shape<LargeShape>();
  if (e == hipSuccess) e = configure_shape<SmallShape>();
  if (e == hipSuccess) e = configure_shape<DeepShape>();
  if (e == hipSuccess) e = configure_shape<PartsShape>();
  return e;
}

hipError_t launch_execute_direct(const ExecuteArgs& args, DirectShape shape, bool tails, int grid, hipStream_t stream) {
  switch (shape) {
    case kDirectLarge: return launch_shape<LargeShape>(args, tails, grid, stream);
    case kDirectSmall: return launch_shape<SmallShape>(args, tails, grid, stream);
    case kDirectDeep: return launch_shape<DeepShape>(args, tails, static_cast<int>(args.n_items), stream);
    default: {   // one workgroup per part of an item; the list is padded to whole rounds of the XCDs
      const int64_t parts = (args.n_items + 7) / 8 * 8 * PartsShape::PARTS;
      return launch_shape<PartsShape>(args, tails, static_cast<int>(parts), stream);
    }
  }
}

}  // namespace cleave
