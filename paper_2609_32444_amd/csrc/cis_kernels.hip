// HIP kernels (gfx950) of the CIS token loss: the base row-kernel variants (CIS weight at
// update ratio 1), the deterministic loss/statistics reduction, and the elementwise weight
// kernel of Algorithm 1. The row kernel itself is in cis_row.h.
#define CIS_EXT false
#include "cis_row.h"
#include "cis_seg.h"

namespace cis {

// ------------------------------------------------------------------------------------------
// Loss and statistics, summed in a fixed order (independent of the row grid). PARTS = false: the
// rows by one workgroup, straight to the results. PARTS = true: workgroup b writes the sums of
// rows [b rows, (b + 1) rows) to parts[b]; cis_finalize_parts_kernel adds those.
// One workgroup is bound by the latency of its loads (13 bytes per row on one compute unit):
// 5.1 us for 256 rows, 9.6 us for 32768, 98 us for 524288.
// ------------------------------------------------------------------------------------------
template <int BLOCK, bool PARTS>
__global__ __launch_bounds__(BLOCK) void cis_finalize_kernel(const FinalizeArgs a) {
  RowStats st{};
  // four rows per thread and step, with 16-byte (4-byte for the flags) loads of the 256-byte
  // aligned workspace arrays; the loop is unrolled so that several steps' loads are in flight
  typedef float f4 __attribute__((ext_vector_type(4)));
  const int64_t t0 = PARTS ? (int64_t)blockIdx.x * a.rows : 0;
  const int64_t te = PARTS && t0 + a.rows < a.T ? t0 + a.rows : a.T;
  const f4* terms4 = reinterpret_cast<const f4*>(a.terms_ws);
  const f4* logk4 = reinterpret_cast<const f4*>(a.logk_ws);
  const f4* exc4 = reinterpret_cast<const f4*>(a.excess_ws);
  const uint32_t* flags4 = reinterpret_cast<const uint32_t*>(a.flags_ws);
#pragma unroll 4
  for (int64_t q = t0 / 4 + threadIdx.x; q < te / 4; q += BLOCK) {
    const f4 tv = terms4[q], lv = logk4[q], ev = exc4[q];
    const uint32_t fv = flags4[q];
#pragma unroll
    for (int e = 0; e < 4; ++e) take_row(st, tv[e], (uint8_t)(fv >> (8 * e)), lv[e], ev[e]);
  }
  for (int64_t t = te / 4 * 4 + threadIdx.x; t < te; t += BLOCK)
    take_row(st, a.terms_ws[t], a.flags_ws[t], a.logk_ws[t], a.excess_ws[t]);
  st = block_stats<BLOCK>(st);
  if (threadIdx.x != 0) return;
  if (PARTS)
    a.parts[blockIdx.x] = st;
  else
    write_stats(a, st);
}

// The sums of the parts: thread i takes parts i, i + BLOCK, ..., then the block's tree.
__global__ __launch_bounds__(kFinalizeParts) void cis_finalize_parts_kernel(const FinalizeArgs a) {
  RowStats st{};
  for (int i = threadIdx.x; i < a.nparts; i += kFinalizeParts) add_stats(st, a.parts[i]);
  st = block_stats<kFinalizeParts>(st);
  if (threadIdx.x == 0) write_stats(a, st);
}

// ------------------------------------------------------------------------------------------
// Algorithm 1 as an elementwise pass over recorded log-probabilities.
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kWeightsBlock) void cis_weights_kernel(const WeightsArgs a) {
  for (int64_t t = (int64_t)blockIdx.x * kWeightsBlock + threadIdx.x; t < a.T;
       t += (int64_t)gridDim.x * kWeightsBlock) {
    float w = 0.f;
    bool trunc = false;
    if (!a.mask || a.mask[t]) {
      const float lt = a.logp_train[t];
      const float delta = lt - a.logp_infer[t];
      const float lam_phi = a.lam * fmaxf(-expm1f(lt), a.kappa);
      trunc = delta > log1pf(lam_phi);
      w = trunc ? 1.0f + lam_phi : expf(delta);
    }
    a.w_out[t] = w;
    if (a.trunc_out) a.trunc_out[t] = trunc ? 1 : 0;
  }
}

// ------------------------------------------------------------------------------------------
// Variant tables
// ------------------------------------------------------------------------------------------
static const RowVariant kBf16Bwd[] = CIS_BWD_TABLE(Bf16);
static const RowVariant kBf16Fwd[] = CIS_FWD_TABLE(Bf16, 18);
static const RowVariant kF32Bwd[] = CIS_BWD_TABLE(F32);
static const RowVariant kF32Fwd[] = CIS_FWD_TABLE(F32, 15);

static const RowVariant kBf16Few[] = CIS_FEW_TABLE(Bf16);
static const RowVariant kF32Few[] = CIS_FEW_TABLE(F32);
const RowVariant* select_row_variant_few(int dtype, int32_t nvec) {
  if (nvec <= kFewMinVec || nvec > kFewMaxVec) return nullptr;
  return &pick_variant(dtype == CIS_BF16 ? kBf16Few : kF32Few, 3, nvec);
}

const RowVariant& select_row_variant(int dtype, bool bwd, int32_t nvec) {
  constexpr int nb = sizeof(kBf16Bwd) / sizeof(kBf16Bwd[0]);
  constexpr int nf = sizeof(kBf16Fwd) / sizeof(kBf16Fwd[0]);
  const RowVariant* t = dtype == CIS_BF16 ? (bwd ? kBf16Bwd : kBf16Fwd) : (bwd ? kF32Bwd : kF32Fwd);
  return pick_variant(t, bwd ? nb : nf, nvec);
}

// Split forward pass. Rows shorter than kSegMinVec vectors stay with the row kernel (one short
// row per workgroup is already a small independent read); longer rows take the first variant
// that covers them with at most kSegMax segments.
constexpr int32_t kSegMinVec = 2048;
#define CIS_SEG(E, B, K, RE)                                                 \
  SegVariant{B, K, (const void*)&cis_seg_kernel<E, B, K, RE, SegUse::kPlain>, \
             (const void*)&cis_seg_kernel<E, B, K, RE, SegUse::kRotated>}
// 128-thread workgroups of 8 vectors each (16 KiB of bf16 logits) measured best at V = 32768,
// 151936 and 262144 among 64-256 threads x 4-16 vectors; longer rows take longer segments.
static const SegVariant kSegBf16[] = {CIS_SEG(Bf16, 128, 8, true), CIS_SEG(Bf16, 128, 16, true),
                                      CIS_SEG(Bf16, 256, 16, true)};
static const SegVariant kSegF32[] = {CIS_SEG(F32, 128, 8, true), CIS_SEG(F32, 128, 16, true),
                                     CIS_SEG(F32, 256, 16, true)};

const SegVariant* select_seg_variant(int dtype, int32_t nvec) {
  if (nvec < kSegMinVec) return nullptr;
  const SegVariant* t = dtype == CIS_BF16 ? kSegBf16 : kSegF32;
  for (int i = 0; i < 3; ++i)
    if ((int64_t)t[i].block * t[i].k * kSegMax >= nvec) return &t[i];
  return nullptr;
}

// Few rows that a compute unit each would work on too long. Fused calls in us, row kernel and
// split (bf16): V = 50257, 32 rows 12.4 and 11.8, 64 rows 12.9 and 13.6; V = 100003, 128 rows 18.8
// and 18.2, 192 rows 20.8 and 23.7; V = 151936, 64 rows 21.0 and 15.4, 96 rows 21.1 and 17.9, 128
// rows 21.6 and 22.6; V = 262144 (LDS slots and streamed ones), 64 rows 35.8 and 17.4, 192 rows
// 52.6 and 47.2, 256 rows 62.7 and 62.3.
static int64_t seg_grad_max_rows(int32_t nvec) {
  return nvec > 19456 ? 192 : (nvec >= 12288 ? 112 : (nvec >= 6144 ? 32 : 0));
}

bool select_seg_grad_variant(int dtype, bool ext, int64_t T, int32_t nvec, SegGradVariant* v) {
  constexpr int kVec = kSegGradBlock * kSegGradK;
  if (T > seg_grad_max_rows(nvec) || nvec > kVec * kSegMax) return false;
  const bool b = dtype == CIS_BF16;
  *v = SegGradVariant{
      kSegGradBlock, kSegGradK,
      b ? (const void*)&cis_seg_kernel<Bf16, kSegGradBlock, kSegGradK, true, SegUse::kGrad>
        : (const void*)&cis_seg_kernel<F32, kSegGradBlock, kSegGradK, true, SegUse::kGrad>,
      ext ? seg_grad_kernel_ext(dtype)
      : b ? (const void*)&cis_seg_grad_kernel<Bf16, kSegGradBlock, kSegGradK, false>
          : (const void*)&cis_seg_grad_kernel<F32, kSegGradBlock, kSegGradK, false>};
  return true;
}

const void* combine_kernel(bool ext, bool lane) {
  if (ext) return combine_kernel_ext(lane);
  return lane ? (const void*)&cis_combine_lane_kernel<false> : (const void*)&cis_combine_kernel<false>;
}

// Clears the row kernel's queue counters ahead of a launch that uses them, where no pre-pass does: a
// kernel rather than a memset, so a captured call holds no memset node.
__global__ __launch_bounds__(64) void cis_queue_reset_kernel(unsigned long long* q) {
  if (threadIdx.x < kRowQueues) q[threadIdx.x * (kQueueStride / sizeof(*q))] = 0ull;
}

const void* finalize_kernel(int block, bool parts) {
  return parts          ? (const void*)&cis_finalize_kernel<256, true>
         : block == 256 ? (const void*)&cis_finalize_kernel<256, false>
                        : (const void*)&cis_finalize_kernel<kFinalizeBlock, false>;
}
const void* finalize_parts_kernel() { return (const void*)&cis_finalize_parts_kernel; }
const void* queue_reset_kernel() { return (const void*)&cis_queue_reset_kernel; }
const void* weights_kernel() { return (const void*)&cis_weights_kernel; }

}  // namespace cis
