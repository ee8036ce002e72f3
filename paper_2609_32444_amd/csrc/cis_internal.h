// Internal interface between the C-ABI entry points (cis_api.cpp) and the HIP kernels
// (cis_kernels.hip, cis_kernels_ext.hip). Not installed; not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/cis.h"
#include "cis_plan.h"

namespace cis {

// Workspace layout (bytes), every array 256-byte aligned:
//   [0, 256)     cis_stats_t, and from 128 the counter by which a kernel's last workgroup knows
//                itself (cleared by the kernel before it)
//   [256, 1280)  the fused pass's row-queue counters, one per 128-byte line; before the rows,
//                the pieces of the responses' log K, where there are several (kSeqPieceSums)
//   terms  float[T]   per-row loss term
//   logk   float[T]   per-row log k (diagnostics)
//   excess float[T]   per-row k - w (diagnostics)
//   wpre   float[T]   weight from the pre-pass (decoupled path); after the rows, the sums of the
//                     statistics' parts (RowStats) where there are several. cis_weights_ex keeps
//                     its workgroups' sums at terms instead, and none of the rows' values.
//   flags  uint8[T]   per-row status bits (kFlag*)
//   pflags uint8[T]   pre-pass bits (kFlagTrunc = acted on)
//   logK   double[n_seq]  per-response log K (sequence operators)
//   part   float2[T * kSegMax]  per-segment (max, exp-sum) of the split passes
//   zy     float[T]           the sampled logit (split passes)
// The last two exist only in the layout of the forward entry points and of the fused pass over
// few rows (`seg`); the other fused calls and the LM-head path do not use them.
constexpr size_t kStatsBytes = 256;
static_assert(sizeof(cis_stats_t) <= kStatsBytes, "the statistics fit their block");
// The row queue: up to kRowQueues counters of 8 bytes, each on a 128-byte line of its own.
// Returning atomics on one line are served one at a time, about 80 M per second on this part,
// which short rows approach (one draw per row); counters on separate lines are served in
// parallel. Short rows use all of them, long rows one (with eight, the long-row workloads ran
// 2-3% slower).
constexpr size_t kDoneOff = 128;   // counter of finished rows, in the same block
static_assert(sizeof(cis_stats_t) <= kDoneOff, "the counter follows the statistics");
constexpr int kRowQueues = 8;
constexpr size_t kQueueOff = kStatsBytes;
constexpr size_t kQueueStride = 128;
constexpr size_t kHeadBytes = kQueueOff + kRowQueues * kQueueStride;
// Sums of pieces of responses that fit the counters' block (which is cleared after their use).
constexpr int kSeqPieceSums = (int)((kHeadBytes - kQueueOff) / sizeof(double));
// Segments per row at most in the split forward pass (the partials per row in the workspace).
constexpr int kSegMax = 32;

// Per-row gradient parameters of the fused LM-head pass (written by the row combine, read by
// the logits product's gradient epilogue): g_j = s exp2(z_j log2(e) - b2) with s = -1 when neg
// (coef > 0), else +1; the sampled column y gets gy; y = -1 for a row without gradient
// (b2 = +inf, gy = 0).
struct GradParams {
  float b2;
  int32_t neg;
  float gy;
  int32_t y;
};

constexpr size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
struct WsLayout {
  size_t terms, logk, excess, wpre, flags, pflags, logK, part, zy, total;
  bool seg;
};
constexpr WsLayout ws_layout(int64_t T, int64_t n_seq, bool seg = false) {
  const size_t f = align_up(4 * (size_t)T, 256), b = align_up((size_t)T, 256);
  WsLayout L{};
  L.terms = kHeadBytes;
  L.logk = L.terms + f;
  L.excess = L.logk + f;
  L.wpre = L.excess + f;
  L.flags = L.wpre + f;
  L.pflags = L.flags + b;
  L.logK = L.pflags + b;
  L.part = L.logK + align_up(8 * (size_t)n_seq, 256);
  L.zy = L.part + (seg ? align_up(8 * (size_t)kSegMax * (size_t)T, 256) : 0);
  L.total = L.zy + (seg ? f : 0);
  L.seg = seg;
  return L;
}
constexpr size_t ws_bytes(int64_t T) { return ws_layout(T, 0).total; }

// LM-head workspace: the loss workspace above, then (256-byte aligned)
//   Q   int[64]   the products' work queues (256 bytes)
//   Z   float[rows, ldz]   the chunk's logits (the default backward only)
//   then per row and 64-column block the pair (max, exp-sum) (float2[rows, ntv]), the sampled
//   logit (float[rows]) and the gradient parameters (GradParams[rows])
//   G   bf16[grows, ldv]   dL/dz of the rows of a dL/dW group (backward)
//   P   float[lm_splits, rows, H]  split-K partials of dL/dh (backward, where it is split)
// with rows = min(T, chunk), grows = min(T, lm_dw_rows(chunk)) and row strides rounded up by
// lm_stride.
constexpr int64_t kLmMaxH = int64_t(1) << 16;
constexpr int64_t kLmMaxChunk = int64_t(1) << 16;
// The products address a 256-row operand tile with 32-bit byte offsets, so operand row strides
// stay below 2^23 elements: V (the contracted length of dL/dh) and ld_h, ld_w up to 2^22.
constexpr int64_t kLmMaxV = int64_t(1) << 22;
constexpr int64_t kLmMaxLd = int64_t(1) << 22;
// Row stride of n elements: whole 128-byte lines of bf16, so that a product's slab rows do not
// straddle two, where that adds at most an eighth; else 16-byte chunks.
inline int64_t lm_stride(int64_t n) { return n >= 512 ? (n + 63) / 64 * 64 : (n + 7) / 8 * 8; }
// Splits of the contraction (V) of dL/dh that the partial buffer holds: with few tiles, as many as
// fill 256 compute units (the buffer is then at most 64 MiB), but no more than the products use
// (gemm_splitk_count: a split keeps kMinSplitLen of the contraction).
constexpr int64_t kMinSplitLen = 512;
inline int64_t lm_splits(int64_t rows, int64_t V, int64_t H) {
  const int64_t tiles = ((rows + 255) / 256) * ((H + 255) / 256);
  const int64_t fill = tiles >= 32 ? 8 : (tiles <= 8 ? 32 : 256 / tiles);
  const int64_t len = V / kMinSplitLen;
  return len < 1 ? 1 : len < fill ? len : fill;
}
// dL/dW is one product per group of consecutive chunks, up to kLmDwRows rows: fewer products
// that accumulate into dL/dW. A group holds whole chunks when chunk is a multiple of 8, otherwise
// it is one chunk (cis_lmhead_loss_bwd states the groups).
constexpr int64_t kLmDwRows = int64_t(1) << 14;
inline int64_t lm_dw_rows(int64_t chunk) {
  if (chunk % 8 != 0 || chunk >= kLmDwRows) return chunk;
  return chunk * (kLmDwRows / chunk);
}
struct LmLayout {
  WsLayout loss;
  int64_t ldz, ldv, ntv, splits;
  size_t z, g, part, queue, total;
  size_t tpart, tzy, tgp;  // the product's (max, exp-sum) pairs, sampled logits, gradient
                           // parameters of the chunk's rows
  bool fused;
};
inline LmLayout lm_layout(int64_t T, int64_t V, int64_t H, int64_t chunk, int64_t n_seq,
                          bool bwd, bool fused) {
  LmLayout M;
  M.fused = fused;
  M.splits = 1;
  M.loss = ws_layout(T, n_seq);
  const int64_t rows = T < chunk ? T : chunk;
  M.ldz = lm_stride(V);
  M.ldv = M.ldz;
  M.ntv = (V + 255) / 256 * 4;  // four 64-column blocks per 256-column tile
  const int64_t grows = T < lm_dw_rows(chunk) ? T : lm_dw_rows(chunk);
  M.queue = align_up(M.loss.total, 256);  // the products' work queues
  M.z = M.queue + 256;
  size_t end = M.z;
  if (!fused) end += align_up((size_t)rows * (size_t)M.ldz * 4, 256);  // the chunk's logits
  M.tpart = end;
  end += align_up((size_t)rows * (size_t)M.ntv * 8, 256);
  M.tzy = end;
  end += align_up((size_t)rows * 4, 256);
  M.tgp = end;
  end += align_up((size_t)rows * sizeof(GradParams), 256);
  M.g = M.part = end;
  if (bwd) {
    end += align_up((size_t)grows * (size_t)M.ldv * 2, 256);
    M.part = end;
    M.splits = rows > 0 ? lm_splits(rows, V, H) : 1;
    if (M.splits > 1) end += align_up((size_t)M.splits * (size_t)rows * (size_t)H * 4, 256);
  }
  M.total = end;
  return M;
}

// Per-row status bits (workspace flags[T]; kFlagTrunc = the operator acted on the row).
enum : uint8_t { kFlagValid = 1, kFlagBadId = 2, kFlagNonFinite = 4, kFlagTrunc = 8 };

// Operator parameters as the kernels see them (cis_params_t minus the loss fields).
struct OpArgs {
  int32_t op;
  float lam, kappa, lo, hi;
};

// Arguments of the row kernels, passed by value.
struct RowArgs {
  const void* logits;       // [T, ld] elements
  void* dlogits;            // [T, ldg] gradient elements (bwd only)
  int64_t row_bytes;        // ld  * sizeof(logit element)
  int64_t grow_bytes;       // ldg * sizeof(gradient element)
  const int64_t* ids;
  const float* logp_infer;
  const float* adv;
  const uint8_t* mask;      // nullable
  float* logp_train_out;    // nullable
  float* w_out;             // nullable
  uint8_t* trunc_out;       // nullable
  float* terms_user;        // nullable
  float* terms_ws;          // workspace terms[T]
  uint8_t* flags_ws;        // workspace flags[T]
  float* logk_ws;           // workspace logk[T]
  float* excess_ws;         // workspace excess[T]
  int64_t T;
  int32_t V;
  int32_t nvec;             // ceil(V / elements per 16-byte vector)
  float lam, kappa, scale;
  // extended kernels only
  OpArgs ops;               // rate-1 path: the operator applied in the epilogue
  const float* logp_old;    // non-null: decoupled path (weight from the pre-pass)
  const float* wpre_ws;     // pre-pass weight[T]
  const uint8_t* pflags_ws; // pre-pass acted bits[T]
  float* eps_out;           // nullable; rate-1 path only (the pre-pass writes it otherwise)
  float clip_low, clip_high;
  // row queue of the row kernel (up to kRowQueues counters, kQueueStride bytes apart), or null
  // where no row comes from it: a workgroup's first three rows are fixed; with n counters in use
  // (see cis_row_kernel), counter c hands out the later rows 3*gridDim.x + c + n*q, q = 0, 1,
  // ... Cleared before the rows by the pre-pass, where it runs, or by queue_reset_kernel.
  unsigned long long* queue;
};

// Rows whose (max, exp-sum) comes in pieces: the split forward pass (cis_seg_kernel) and the
// fused LM-head pass (the logits product's epilogue), folded by cis_combine_kernel.
struct SegArgs {
  float2* part;     // [T * stride] (max, exp-sum without the sampled logit) per piece
  float* zy;        // [T] the sampled logit
  int32_t nseg;     // pieces per row (<= stride)
  int32_t segvec;   // 16-byte vectors per segment (split forward pass)
  int64_t stride;   // pieces per row in `part`
  GradParams* gp;   // [T] nullable: gradient parameters for the fused LM-head pass
  uint32_t* done;   // rows whose outputs are stored (the fused pass over few rows)
  int32_t rot;      // seg_rotation() (split forward pass)
};
// Workgroup b runs on XCD b % 8, so the segment at a given place of the row meets the same XCD again
// after 8 / gcd(nseg, 8) rows: one more place of rotation from then on. None (-1) for an odd nseg,
// which visits every XCD by itself, and for equal segments: there the plain order is the faster one
// (16384 rows of V = 151936 782 us against 798, V = 32768 171 against 178). Nor for four segments
// with the last one less than a quarter full (V = 24657 172.5 us against 175.8; from V = 26214 on the
// two are within 1%, and float32 rows of V = 14336 gain: 85.7 and 79.8).
inline int32_t seg_rotation(int32_t nseg, int32_t segvec, int32_t nvec) {
  const int32_t last = nvec % segvec;
  if (nseg % 2 != 0 || last == 0 || (nseg == 4 && 4 * last < segvec)) return -1;
  return nseg % 8 == 0 ? 0 : nseg % 4 == 0 ? 1 : 2;
}
constexpr int kCombineBlock = 256;
constexpr int kSegGradBlock = 128, kSegGradK = 8;   // 16 KiB of logits per workgroup
// A compiled segment kernel: `block` threads with K 16-byte vectors each, so block * K vectors
// per segment. SegUse is what it is for (see cis_seg_kernel).
enum class SegUse { kPlain, kRotated, kGrad };
struct SegVariant {
  int block, k;
  const void *fn, *rotated;   // segments in order, and rotated (seg_rotation)
};
// The segment kernel for rows of `nvec` vectors, or nullptr when the row kernel serves them
// better (short rows) or they need more than kSegMax segments of the largest variant.
const SegVariant* select_seg_variant(int dtype, int32_t nvec);
// The fused pass over few long rows: cis_seg_kernel (`fn`), then cis_seg_grad_kernel (`grad`) over
// the same segments. select_seg_grad_variant returns false, and sets nothing, when the row kernel
// serves such a call better.
struct SegGradVariant {
  int block, k;
  const void *fn, *grad;
};
bool select_seg_grad_variant(int dtype, bool ext, int64_t T, int32_t nvec, SegGradVariant* v);
const void* seg_grad_kernel_ext(int dtype);
// lane: one lane per row (rows of at most kSegMax pieces), else one wave per row
const void* combine_kernel(bool ext, bool lane);
const void* combine_kernel_ext(bool lane);

// Sums of the statistics over some rows (cis_stats.h).
struct alignas(64) RowStats {
  double loss, excess;
  float max_logk;
  long long valid, bad_id, nonfinite, acted;
};

struct FinalizeArgs {
  const float* terms_ws;
  const uint8_t* flags_ws;
  const float* logk_ws;
  const float* excess_ws;
  int64_t T;
  cis_stats_t* stats;
  float* loss_out;          // nullable
  cis_stats_t* stats_copy;  // nullable: a second copy of the statistics (caller's memory)
  RowStats* parts;          // sums of the rows' parts, where they are summed apart
  int64_t rows;             // rows per part
  int32_t nparts;
};
// Rows that one workgroup of 256, or of kFinalizeBlock, sums at once; more are summed in parts of
// at least kFinalizeRows rows, at most kFinalizeParts of them.
constexpr int64_t kFinalizeSmall = 1024;
constexpr int64_t kFinalizeOne = 16384;
constexpr int64_t kFinalizeRows = 4096;
constexpr int kFinalizeParts = 256;

struct WeightsArgs {
  const float* logp_train;
  const float* logp_infer;
  const uint8_t* mask;      // nullable
  float* w_out;
  uint8_t* trunc_out;       // nullable
  int64_t T;
  float lam, kappa;
};

// Per-response sum of log k over valid tokens (sequence operators).
struct SeqSumArgs {
  const float* logp_p;
  const float* logp_q;
  const uint8_t* mask;      // nullable
  const int64_t* ids;       // nullable (weights path: validity is the mask alone)
  const int64_t* offsets;   // [n_seq + 1]
  double* logK;             // [n_seq * pieces]
  int64_t T, n_seq;
  int32_t V;
  int32_t pieces;           // parts of a response that are summed apart
};

// Per-token weights of an operator from recorded log-probabilities: the decoupled path's
// pre-pass and cis_weights_ex.
struct PrepassArgs {
  const float* logp_p;
  const float* logp_q;
  const uint8_t* mask;      // nullable
  const int64_t* ids;       // nullable
  const int64_t* offsets;   // sequence operators
  const double* logK;       // sequence operators: [n_seq * pieces]
  int32_t pieces;           // parts of a response's log K, added in order
  OpArgs ops;
  int64_t T, n_seq;
  int32_t V;
  float* w_out;             // nullable
  uint8_t* acted_out;       // nullable
  float* eps_out;           // nullable
  float* wpre_ws;           // nullable (loss path)
  uint8_t* pflags_ws;       // nullable (loss path)
  float* logk_ws;           // nullable (loss path), as excess_ws
  float* excess_ws;
  RowStats* parts;          // nullable: weights path: each workgroup's statistics
  unsigned long long* queue;  // nullable: row-queue counters to clear (loss path)
};

// A compiled row-kernel variant: BLOCK threads per workgroup, NV register-resident 16-byte
// vectors per thread.
struct RowVariant {
  int block;
  int nv;                   // slots held in registers
  int nl;                   // further slots held in LDS (0: the last slot sits in a register)
  const void* fn;           // __global__ function (for hipLaunchKernel / occupancy queries)
};

// Picks the variant for `nvec` 16-byte vectors per row; dtype is CIS_BF16 or CIS_F32. The
// extended variants carry the operator family and the decoupled path in their epilogue.
const RowVariant& select_row_variant(int dtype, bool bwd, int32_t nvec);
const RowVariant& select_row_variant_ext(int dtype, bool bwd, int32_t nvec);

// 256 or kFinalizeBlock threads; 256 with parts
const void* finalize_kernel(int block, bool parts);
// The fused variant for calls of few rows per workgroup of the variant above that the chip holds at
// once (at most few_rounds, and more than one row per CU), or null where there is none (see
// CIS_FEW_TABLE). With a mask no more than 4: a workgroup's first three rows are fixed, and over
// more rounds than that the smaller blocks, which are more, leave too few rows to the queue to make
// up for masked ones (half of the rows masked: V = 32768, 3001 rows 65.9 us with the ladder's blocks
// and 74.9 with these, 4096 rows 86.6 and 93.1; V = 50257, 1536 rows 62.1 and 64.4; V = 65536, 1300
// rows 60.8 and 65.6; up to 4 rounds these are the faster ones or equal, masked or not).
inline int64_t few_rounds(int32_t nvec, bool masked) {
  if (nvec > 2048 && nvec <= 3584) return 0;
  return masked || nvec <= 2048 ? 4 : nvec > 4096 ? 6 : 16;
}
const RowVariant* select_row_variant_few(int dtype, int32_t nvec);
const RowVariant* select_row_variant_few_ext(int dtype, int32_t nvec);

const void* finalize_parts_kernel();                 // kFinalizeParts threads
const void* queue_reset_kernel();
const void* weights_kernel();
const void* seq_sum_kernel(int threads);  // 64 (a wave per response) or kSeqBlock
const void* prepass_kernel();
constexpr int kFinalizeBlock = 1024;
constexpr int kWeightsBlock = 256;

}  // namespace cis
