// Launch interface between the C-ABI layer and the HIP kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "plan_internal.h"

namespace cleave {

// Most members a grouped launch (one table entry per member) can have.
constexpr int kMaxGroup = 8;

// Where batch member g's matrix starts, as an element offset from the base
// pointer.  Strided batch (batch_inner > 0): member o * batch_inner + i at
// o * outer + i * inner.  Grouped launch (n_group > 0): member g at table[g].
// Plain plans have one member at offset 0.
struct MemberOffsets {
  int64_t outer, inner;
  int64_t table[kMaxGroup];
};

struct BatchShape {
  uint32_t batch_inner;
  uint32_t n_group;
};

__host__ __device__ inline int64_t member_offset(const MemberOffsets& at, BatchShape b, uint32_t gemm_id) {
  if (b.n_group != 0) return at.table[gemm_id];
  if (b.batch_inner == 0) return 0;
  const uint32_t o = gemm_id / b.batch_inner;
  return static_cast<int64_t>(o) * at.outer + static_cast<int64_t>(gemm_id - o * b.batch_inner) * at.inner;
}

struct ExecuteArgs {
  const WorkItem* items;      // device work items of one tile class (self-contained records)
  int64_t n_items;
  const void* A;
  const void* B;
  int64_t lda, ldb;           // elements
  int transA, transB;
  float* partials;
  // Batched plans: task.gemm_id selects the member's operands (and, in
  // assemble mode, its output) through these offsets.
  BatchShape batch;
  MemberOffsets a_at, b_at, c_at;
  // Assemble mode (C != nullptr): blocks go straight to their place in the
  // output matrix (fp32, or bf16 when c_bf16 != 0) instead of `partials`.
  void* C;
  int64_t ldc;
  int c_bf16;
  // Direct kernel's large shape only: items whose chunk starts below this k leave through
  // non-temporal stores (streamed_below in api.cpp).
  uint32_t stream_below_k;
  // General kernel only: extent of the logical operands (loads stay inside them)
  // and the workgroup tiles per work item (filled in at the launch).
  int64_t M, N, K;
  int parts_m, parts_n;
  // Direct kernel only, shapes with several items per workgroup.  Null:
  // workgroup b takes items b, b + grid, ...  Otherwise grid + 1 entries:
  // workgroup b takes items [wg_ranges[b], wg_ranges[b + 1]).
  const uint32_t* wg_ranges;
};

// Bytes of the Infinity Cache: what is written last, up to that much, is still
// there when the next launch reads it.
constexpr int64_t kCacheBytes = int64_t{256} << 20;

// Whether the direct kernel streams an assembled output of `bytes` (streamed_below in
// api.cpp).  A batch from the cache's size on: scores of 1024 x 1024 x members into bf16, us,
// plain / streamed, the launch alone, with a softmax, an update in place, the largest value
// of all behind it:
//   134 MB    33 / 33     136 / 148    71 / 76     89 / 110
//   168 MB    39 / 39     158 / 191    84 / 89    104 / 131
//   201 MB    43 / 44     216 / 224    98 / 104   121 / 154
//   235 MB    72 / 51     267 / 257   137 / 136   164 / 176
//   268 MB    83 / 61     301 / 287   158 / 158   209 / 198
//   336 MB   102 / 73     371 / 357   216 / 196   294 / 254
//   537 MB   157 / 112    580 / 564   338 / 316   453 / 425
// A reader that does little else still loses 7 % just below the cache's size.  A single
// output, all of it in one order, is held a little longer: alone, with a product into
// another matrix, in place, the largest value, K = 128 and 512, 268 MB of fp32 50 / 54,
// 155 / 149, 131 / 133, 119 / 135 and 83 / 85, 180 / 178, 161 / 164, 161 / 164, of bf16 60 / 55,
// 164 / 157, 139 / 134, 170 / 198 and 127 / 124, 221 / 220, 201 / 198, 239 / 260; 302 MB of fp32
// 57 / 64, 175 / 167, 147 / 149, 162 / 151 and 95 / 94, 212 / 203, 186 / 181, 198 / 182, of bf16
// 64 / 65, 186 / 170, 159 / 152, 230 / 222 and 146 / 144, 250 / 244, 227 / 225, 295 / 289; 361 MB
// of bf16 79 / 75, 216 / 202, 189 / 182, 288 / 261.  So those from an eighth more on.  (A launch
// of K up to 128 that only overwrites its own output again loses 11 to 19 % at 302 MB.)
inline bool streamed_output(int64_t bytes, bool batched) {
  return bytes >= (batched ? kCacheBytes : kCacheBytes / 8 * 9);
}

// Workgroup tile of the general execute kernel: 128 x 128, 64 x 64, 256 x 256
// (only for bf16 work items of the large class with both operands K-contiguous), or
// the quarters of the 64 x 64 one (32 x 32, only fp32).  kTileWide4: 128 x 128 in four waves.
// kTileLone: 64 x 64, reading a K step ahead.
enum ExecuteTile : int { kTileWide = 0, kTileNarrow = 1, kTileHuge = 2, kTileQuarter = 3, kTileWide4 = 4, kTileLone = 5 };

// Whether a list of `items` 128 x 128 tiles runs in four waves of 64 x 64 each instead of eight
// of 32 x 64.  Eight read half as much again from LDS per product and hide a workgroup's start
// and end, a wait for operands and a round that is not full; over several rounds the chip is
// full anyway.  bf16 with two K-contiguous operands (whose wave tiles of 64 x 64 read the
// least), from three rounds of the CUs on; TN, whose transpose reads are the dearest, from
// seven on with chunks beyond 256.  us, four waves / eight, each running by itself:
//   elements         33            515            1023           2047           4095
//   NT  1024     17.9 / 18.8    37.8 / 38.3    46.7 / 47.6    81.7 / 83.5   153 / 154
//       1155                    44.3 / 45.0    55.2 / 56.8    97.0 / 97.4   182 / 184
//       2048     29.1 / 31.4    70.0 / 74.0    90.0 / 91.0    160 / 161     299 / 302
//       4096     51.4 / 55.7    134 / 144      178 / 180      316 / 320     595 / 609
//   TN  1024     16.9 / 16.4    36.5 / 35.1    55.0 / 55.6    97.0 / 98.8   181 / 192
//       1155                    43.0 / 41.5    66.0 / 66.0    119 / 118     223 / 220
//       2048     28.5 / 28.4    67.1 / 67.8    107 / 111      192 / 198     361 / 369
//       4096     51.3 / 50.1    134 / 135      216 / 221      383 / 394     739 / 755
// NN and TT are 1 % slower to 6 % faster in eight but for 4096 items of 515 (134 / 136, 133 /
// 136).  Between launches of other kernels eight gain up to 4 % more with long chunks.
// fp32 from four rounds on with up to 128 elements, but for NN, which changes side at every
// length (.962 to 1.021); time of eight over four's, NT, TN, TT: 1280 items of 64 1.045,
// 1.053, 1.043, of 128 1.020, 1.012, 1.020, of 192 1.002, 1.012, 1.002; 4096 items of 64 1.036,
// 1.036, 1.029, of 128 1.005, 1.011, 1.001, of 512 .992, .990, .963; 1024 of 64 .997, 1.018, .985.
inline bool four_waves(int dtype, int transA, int transB, int64_t items, const ListShape& list, int cus) {
  if (dtype == CLEAVE_BF16)
    return transA != transB && (transB ? items > int64_t{3} * cus : items > int64_t{7} * cus && list.longest > 256);
  return (transA || transB) && items > int64_t{4} * cus && list.longest <= 128;
}
// An operand with rows shorter than 16 bytes is loaded one element at a time
// (64 x 64 tile, whatever `tile`); the other one still takes 16-byte loads.
struct GeneralLoads {
  ExecuteTile tile;
  bool a_elements, b_elements;
  ListShape list;
  int cus;   // of the device
};

// Workgroup tiles along an edge of the work items of a list whose blocks have at most
// `extent` rows (columns) there: an item of small blocks is not cut into tiles that hold
// nothing.  (Those leave at once, but the workgroups are dealt to the CUs in turn, and
// every other one, or three of four, being empty left half or three quarters of the
// CUs without work.)  fp32 in 64 x 64 tiles, 1024 of K, us, layouts NN, NT, TN, all tiles of
// the items / these: 288 blocks of 64 x 64 79.2 / 36.2, 77.9 / 33.6, 79.4 / 36.1, 300 of 64 x 128
// 80.4 / 54.0, 79.0 / 50.9, 80.7 / 52.7.
inline int parts_along(uint32_t extent, int item, int tile) {
  const int most = extent < static_cast<uint32_t>(item) ? static_cast<int>(extent) : item;
  return (most + tile - 1) / tile;
}

// Workgroups of a general launch over `blocks` workgroup tiles, of which the chip holds
// `resident` at a time.  Between one round and two, the workgroups that fit take their
// second tile themselves: number b's is on the CU of number b - resident, so a second
// round of half as many is spread over all CUs (workgroups are dealt to the CUs in
// turn).  Left to the dispatcher, the first CUs to finish get a full second round and
// the others none.  us, dispatcher / taken, layouts NN, NT, TN: bf16, 128 x 128, 768 tiles
// of 10 steps 36.1 / 35.1, 33.2 / 33.3, 32.2 / 32.2, of 3 17.9 / 17.2, 17.6 / 16.3, 19.2 / 17.4,
// 544 of 16 34.3 / 32.6, 32.5 / 31.3, 40.1 / 39.1; fp32, 128 x 128, 768 of 32 187 / 183, 186 /
// 184, 188 / 185; 64 x 64, 1152 of 32 84.3 / 81.1, 83.0 / 80.3, 84.5 / 81.4, of 8 27.8 / 26.5,
// 29.0 / 26.1, 29.0 / 26.7, 1536 of 32 the same, 1792 of 32 116 / 116, 125 / 114, 118 / 117.
//   `taken_up_to` (second_tiles_taken_up_to): two rounds for 64 x 64; for 128 x 128 one and a
// half, two with short chunks, up to 256 elements: longer ones lose there.  bf16, 832 tiles of 8
// steps 32.8 / 34.7, 35.7 / 37.5, 33.4 / 34.5, of 32 81 / 84, 76 / 79, 89 / 93, 1024 of 32 87 / 90,
// 82 / 84, 94 / 99, of 3 22.1 / 21.4, 21.9 / 20.8, 23.6 / 22.1; fp32, 1024 of 32 246 / 247, 243 /
// 243, 248 / 250, of 8 72.5 / 70.7, 72.6 / 70.9, 74.2 / 72.3.  Behind two rounds the finish
// times are spread anyway: bf16, 1920 tiles of 4 steps 45.6 / 46.2, 4095^3 219 / 226, fp32
// 4096^3 1007 / 1016.
//   Nothing (0) without equal chunks: a fixed pairing can put two long ones on one workgroup,
// where the dispatcher hands the next tile to whoever is done.  Tiles of 128 with one,
// two or four splits at random, dispatcher / taken: fp32, 1536 x 1536 x 2048 94.2 / 115, 91.9 /
// 114, 93.0 / 115, 1536 x 1024 x 4096 (up to eight) 142 / 161, 140 / 160, 142 / 161; bf16 with
// unaligned rows, 2048 x 2048 x 2048 36.2 / 43.6, 37.5 / 43.8, 35.9 / 43.7, one or two, 3072 x
// 3072 x 512 25.7 / 28.2, 26.1 / 28.4, 26.6 / 28.9.
inline int general_workgroups(int64_t blocks, int64_t resident, int64_t taken_up_to) {
  if (blocks > resident && blocks <= taken_up_to) return static_cast<int>(resident);
  constexpr int64_t kMaxGrid = int64_t{1} << 20;   // the kernel loops beyond that
  return static_cast<int>(blocks < kMaxGrid ? blocks : kMaxGrid);
}
// Whether a list of `items` work items that runs in 64 x 64 tiles runs in the form that reads a K step
// ahead: at most one workgroup per CU, and eight steps or more in the longest chunk (both
// sides beside the form, Lone in execute.hip).
inline bool runs_lone(int dtype, int tile_class, int64_t items, const ListShape& list, int cus) {
  const int64_t workgroups = (items + 7) / 8 * 8 * parts_along(list.rows, tile_rows(tile_class), 64) *
                             parts_along(list.cols, tile_cols(tile_class), 64);
  return workgroups <= cus && list.longest > (dtype == CLEAVE_BF16 ? 7u * 64 : 7u * 32);
}
inline int64_t second_tiles_taken_up_to(int64_t resident, int tile, const ListShape& list) {
  if (!list.equal()) return 0;
  return tile == 64 || list.longest <= 256 ? 2 * resident : resident / 2 * 3;
}

// Enqueues the general execute kernel over work items of one tile class: any
// element type, size and alignment.
hipError_t launch_execute(const ExecuteArgs& args, int dtype, int tile_class, const GeneralLoads& how,
                          hipStream_t stream);

// Shape of the direct kernel: one for the large class, three for the small one
// (128 x 128 items, two workgroups per CU; the same with twice the ring, one per
// CU and item; 64 x 64 parts of an item, one workgroup each).  The bits do not depend on
// it.
enum DirectShape : int { kDirectLarge = 0, kDirectSmall = 1, kDirectDeep = 2, kDirectParts = 3 };
// Workgroups one CU holds at a time.
constexpr int direct_workgroups_per_cu(DirectShape shape) {
  return shape == kDirectLarge || shape == kDirectDeep ? 1 : 2;
}
// Enqueues the bf16 direct-to-LDS execute kernel.  The caller has checked the
// 16-byte load conditions.  `tails`: the chunk length of some item may be no
// multiple of kDirectKStep elements (false where one is: its last step reads too far).  `grid` persistent workgroups (kDirectDeep and
// kDirectParts: one workgroup per item or part, whatever `grid`).
hipError_t launch_execute_direct(const ExecuteArgs& args, DirectShape shape, bool tails, int grid, hipStream_t stream);

// Raises the dynamic-LDS limit of every execute kernel on the current device
// (needed once per device and process, before the first launch).
hipError_t configure_execute_kernels();
hipError_t configure_execute_direct_kernels();

// ---- work-item lists of subset launches ---------------------------------------
// One entry per re-issued task: which task, and where its work items go.  The
// entries travel in the kernel arguments, so the launch needs no host buffer,
// no copy and nothing the caller could not capture into a HIP graph.
struct SubsetEntry {
  uint32_t task;   // index into the task table
  uint32_t dst;    // index of the task's first work item in `out`
};
constexpr int kSubsetEntriesPerLaunch = 480;
struct ExpandArgs {
  const cleave_task* tasks;
  WorkItem* out;
  uint32_t n_entries;
  uint32_t fine;             // every block cut into small-class sub-tiles
  SubsetEntry entries[kSubsetEntriesPerLaunch];
};
static_assert(sizeof(ExpandArgs) <= 4096, "kernel arguments stay within 4 KB");
// out[dst + sub] = work item `sub` of entries[e].task, for every entry.
hipError_t launch_expand_subset(const ExpandArgs& args, hipStream_t stream);

// Enqueues the kernel that writes the aggregation's records: one per run of every tile.
hipError_t launch_expand_reduce(const cleave_task* tasks, const ReduceTile* tiles, int64_t n_tiles, ReduceItem* out,
                                hipStream_t stream);

struct ReduceArgs {
  const ReduceItem* items;
  int64_t n_items;
  const float* partials;
  void* C;
  int64_t ldc;                // elements
  BatchShape batch;           // as in ExecuteArgs; offsets apply to C
  MemberOffsets c_at;
};

// Enqueues the aggregation kernel.  `vec` selects the float4 path.
hipError_t launch_reduce(const ReduceArgs& args, int out_dtype, bool vec, int grid,
                         hipStream_t stream);

// Aggregation with a residual added: C = sum of partials + R; R has C's
// element type, leading dimension and batch strides.
hipError_t launch_reduce_residual(const ReduceArgs& args, const void* R, int out_dtype, bool vec,
                                  int grid, hipStream_t stream);

// Aggregation feeding an Adam update of the weight whose gradient the sum is
// (ReduceArgs::C unused; w, m, v, w_bf16 share ldc and the batch strides).
struct AdamArgs {
  float* w;
  float* m;
  float* v;
  uint16_t* w_bf16;   // may be null
  float lr, beta1, beta2, eps, weight_decay;
  float inv_bias1, inv_bias2;   // 1 / (1 - beta^step)
};
hipError_t launch_reduce_adam(const ReduceArgs& args, const AdamArgs& h, bool vec, int grid,
                              hipStream_t stream);
// Grouped form: h holds member 0's arrays, `at` the element offsets of member
// g's arrays from them (ReduceArgs::c_at must be all zero: every array has its
// own table).
struct AdamGroupOffsets {
  int64_t w[kMaxGroup], m[kMaxGroup], v[kMaxGroup], w_bf16[kMaxGroup];
};
hipError_t launch_reduce_adam_grouped(const ReduceArgs& args, const AdamArgs& h, const AdamGroupOffsets& at,
                                      bool vec, int grid, hipStream_t stream);

// ---- returned-block check ---------------------------------------------------

// Projection of a stored operand onto a weight vector, once per segment:
//   out[seg][k]     = sum_{i in seg} x(i, k) * w[seg.start + i]
//   out_abs[seg][k] = sum_{i in seg} |x(i, k)| * |w[seg.start + i]|
// for k in [0, K).  reduce_contiguous = false: x(i, k) = src[i * ld + k] (the
// summed index strides, k is contiguous); true: x(i, k) = src[k * ld + i].
// Batched plans: the projection is made once per (member, segment); member g's
// operand starts member_offset(at, batch, g) elements after src, its weights
// g * w_stride entries after w, and its outputs follow member g-1's (index
// (g * n_segs + seg) * K + k).  Plain plans: n_members = 1, offsets zero.
struct ProjectArgs {
  const void* src;
  int64_t ld;               // elements
  const Segment* segs;
  int n_segs;
  const float* w;
  double* out;
  double* out_abs;
  int64_t K;
  int n_members;
  int64_t w_stride;
  BatchShape batch;
  MemberOffsets at;
};

// item_sums[item] = sum_{rows of the item} r[m0 + i] * sum_j P[i][j] * s[n0 + j].
// Batched plans (batched != 0): the item's gemm_id selects the member's probe vectors,
// r_stride / s_stride entries apart.
struct BilinearArgs {
  const VerifyItem* items;
  int64_t n_items;
  const float* partials;
  const float* r;
  const float* s;
  double* item_sums;
  int batched;
  int64_t r_stride, s_stride;
};

// The two projections and the bilinear items in one launch.  a_contig /
// b_contig: the summed index of that operand is the contiguous one.  `vec`
// selects 16-byte loads for all three jobs (caller has checked alignment and
// divisibility for all of them).
struct VerifyPassArgs {
  ProjectArgs A, B;
  BilinearArgs bil;
};
hipError_t launch_verify_pass(const VerifyPassArgs& args, int dtype, bool a_contig, bool b_contig,
                              bool vec, hipStream_t stream);

// The same pass with the aggregation folded in: a run of rows of a tile is
// taken for all of the tile's splits at once (the S blocks of a tile are
// adjacent, each m_len * n_len elements), so that every partial element is
// read once for both its check and the sum.  The runs are shorter than the
// bilinear items of the separate pass (the pass also writes; short items
// measured 15-25 % faster).  The sum for split s goes to
// item_sums[item.slot + s * item.slot_step]; C gets the left fold
// ((P0 + P1) + ...) + P_{S-1} in fp32.  Splits per tile: at most kMaxFusedSplits.
constexpr int kMaxFusedSplits = 8;
struct AggregateArgs {
  const VerifyItem* items;
  int64_t n_items;
  void* C;
  int64_t ldc;                    // elements
  int out_bf16;
  int stream;                     // fp32 sums leave through non-temporal stores
};
// Whether a check of `partials` elements writes its fp32 sum of `outputs` elements
// with non-temporal stores: where the pass alone gains and nobody who reads the sum next
// loses.  A sum that fits the Infinity Cache is still there for its reader, unless it was
// streamed; one that does not pushes its own first part out again.  us, plain / streamed,
// blocks not in any cache: the pass alone, with a product into another matrix, an
// update in place, a sum over all of it behind it:
//   67 MB in 4 splits    67 / 70     87 / 94     87 / 93     87 / 97
//  134 MB in 4          124 / 129   181 / 180   165 / 171   157 / 172
//  168 MB in 2          105 / 98    166 / 162   157 / 151   152 / 149     in 4 166 / 155   227 / 217   215 / 209   206 / 205
//         in 5          202 / 191   267 / 257   259 / 247   248 / 243     in 8 299 / 290   362 / 352   346 / 343   331 / 341
//  180 MB in 2          111 / 104   177 / 172   168 / 163   160 / 158     in 4 178 / 165   242 / 231   234 / 224   220 / 218
//         in 5          213 / 202   284 / 273   276 / 266   262 / 259     in 8 322 / 309   386 / 376   376 / 367   357 / 363
//  189 MB in 2          116 / 111   197 / 188   187 / 177   177 / 169     in 4 192 / 181   260 / 255   250 / 249   235 / 241
//  201 MB in 2          122 / 116   199 / 193   186 / 187   174 / 175     in 4 195 / 186   268 / 260   260 / 256   243 / 244
//  235 MB in 2          143 / 135   227 / 222   209 / 219   193 / 201     in 4 230 / 217   305 / 301   296 / 300   272 / 284
//  268 MB in 2          169 / 158   263 / 255   249 / 259   244 / 239     in 4 259 / 253   348 / 347   343 / 351   327 / 331
//         in 8          461 / 465   547 / 560   551 / 565   528 / 542
//  302 MB in 1          137 / 118   242 / 227   241 / 230   222 / 209     in 4 295 / 272   391 / 383   405 / 388   369 / 361
//         in 5          351 / 329   451 / 439   464 / 445   432 / 419     in 8 540 / 517   632 / 636   655 / 643   600 / 612
//  336 MB in 2          211 / 185   322 / 308   332 / 315   301 / 285     in 4 326 / 298   433 / 419   454 / 427   409 / 396
//  361 MB in 5          425 / 398   538 / 530   563 / 539   506 / 505     in 7 577 / 544   686 / 680   711 / 691   647 / 655
//  453 MB in 5          536 / 504   679 / 668   703 / 677   640 / 636     in 8 816 / 782   952 / 954   986 / 964   902 / 920
//  537 MB in 4          529 / 472   693 / 662   723 / 676   651 / 624     in 8 972 / 911  1135 /1119  1171 /1135  1075 /1075
// The linear layer's three GEMMs one behind the other (180, 67 and 180 MB in 4 splits; the
// 67 MB stay plain) 523 / 485.
inline bool streamed_sum(int64_t outputs, int64_t partials) {
  const int64_t mib = outputs >> 18;   // whole MiB of fp32
  return partials <= 5 * outputs && ((mib >= 160 && mib < 176) || mib >= 288);
}

struct VerifyReducePassArgs {
  ProjectArgs A, B;
  BilinearArgs bil;
  AggregateArgs agg;
};
hipError_t launch_verify_reduce_pass(const VerifyReducePassArgs& args, int dtype, bool a_contig,
                                     bool b_contig, bool vec, hipStream_t stream);

// Per task: lhs = sum of its item sums (ascending), rhs = sum_k U[k] V[k] and
// scale = sum_k |U|[k] |V|[k] over the task's chunk, accept = |lhs - rhs| <= tol * scale.
struct VerdictArgs {
  const cleave_task* tasks;
  int64_t n_tasks;
  const uint32_t* task_row_seg;
  const uint32_t* task_col_seg;
  const uint32_t* task_first_item;
  const double* item_sums;
  const double* U;
  const double* U_abs;
  const double* V;
  const double* V_abs;
  int64_t K;
  int batched;          // task.gemm_id selects the member's projections
  int n_row_segs, n_col_segs;
  double tol;
  double* lhs;      // any of lhs, rhs, scale may be null
  double* rhs;
  double* scale;
  int32_t* accept;
};
hipError_t launch_verdict(const VerdictArgs& args, hipStream_t stream);

}  // namespace cleave
