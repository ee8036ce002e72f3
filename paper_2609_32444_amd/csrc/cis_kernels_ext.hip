// HIP kernels (gfx950) of the operator family and the decoupled PPO-clip path: the extended
// row-kernel variants (cis_row.h with EXT), the per-response log K of the sequence operators,
// and the per-token weight pass over recorded log-probabilities (cis_weights_ex, and the
// decoupled path's pre-pass).
#define CIS_EXT true
#include "cis_row.h"
#include "cis_seg.h"

namespace cis {

static const RowVariant kBf16BwdExt[] = CIS_BWD_TABLE(Bf16);
static const RowVariant kBf16FwdExt[] = CIS_FWD_TABLE(Bf16, 18);
static const RowVariant kF32BwdExt[] = CIS_BWD_TABLE(F32);
static const RowVariant kF32FwdExt[] = CIS_FWD_TABLE(F32, 15);
static const RowVariant kBf16FewExt[] = CIS_FEW_TABLE(Bf16);
static const RowVariant kF32FewExt[] = CIS_FEW_TABLE(F32);
const RowVariant* select_row_variant_few_ext(int dtype, int32_t nvec) {
  if (nvec <= kFewMinVec || nvec > kFewMaxVec) return nullptr;
  return &pick_variant(dtype == CIS_BF16 ? kBf16FewExt : kF32FewExt, 3, nvec);
}

const RowVariant& select_row_variant_ext(int dtype, bool bwd, int32_t nvec) {
  constexpr int nb = sizeof(kBf16BwdExt) / sizeof(kBf16BwdExt[0]);
  constexpr int nf = sizeof(kBf16FwdExt) / sizeof(kBf16FwdExt[0]);
  const RowVariant* t = dtype == CIS_BF16 ? (bwd ? kBf16BwdExt : kBf16FwdExt)
                                          : (bwd ? kF32BwdExt : kF32FwdExt);
  return pick_variant(t, bwd ? nb : nf, nvec);
}

__device__ __forceinline__ bool token_valid(const uint8_t* mask, const int64_t* ids, int V,
                                            int64_t t) {
  if (mask && mask[t] == 0) return false;
  if (ids) {
    const int64_t y = ids[t];
    return y >= 0 && y < (int64_t)V;
  }
  return true;
}

// ------------------------------------------------------------------------------------------
// Sequence operators (Table tab:baselines, Seq-TIS / Seq-MIS): log K of every response, the
// float64 sum of log k = l_p - l_q over its valid tokens. A response is summed by one wave
// (short responses) or by `pieces` workgroups of THREADS threads, each over an equal part of
// its tokens; threads take the tokens in a fixed stride and reduce in a fixed tree, and the
// pieces are added in order by their reader, so K is deterministic. The sum is bound by the
// latency of its loads: kSeqUnroll tokens of a thread are in flight at once, and 64 responses of
// 8192 tokens took 68.6 us with one wave per response and one token in flight.
// ------------------------------------------------------------------------------------------
constexpr int kSeqUnroll = 4;
template <int THREADS>
__global__ __launch_bounds__(THREADS <= 64 ? 4 * THREADS : THREADS) void cis_seq_sum_kernel(
    const SeqSumArgs a) {
  constexpr int NW = THREADS / 64;
  const int lane = threadIdx.x % THREADS;
  const int64_t u = NW == 1 ? (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6) : (int64_t)blockIdx.x;
  const int64_t s = u / a.pieces, piece = u % a.pieces;
  if (s >= a.n_seq) return;  // whole waves (NW == 1) or workgroups leave together
  int64_t b = a.offsets[s], e = a.offsets[s + 1];
  b = b < 0 ? 0 : (b > a.T ? a.T : b);
  e = e < b ? b : (e > a.T ? a.T : e);
  const int64_t len = (e - b + a.pieces - 1) / a.pieces;
  b = b + piece * len < e ? b + piece * len : e;
  e = b + len < e ? b + len : e;
  double acc = 0.0;
  for (int64_t t0 = b + lane; t0 < e; t0 += kSeqUnroll * THREADS) {
    float lp[kSeqUnroll], lq[kSeqUnroll];
    bool ok[kSeqUnroll];
#pragma unroll
    for (int k = 0; k < kSeqUnroll; ++k) {
      const int64_t t = t0 + k * THREADS;
      ok[k] = t < e;
      const int64_t tc = ok[k] ? t : t0;
      ok[k] = ok[k] && token_valid(a.mask, a.ids, a.V, tc);
      lp[k] = a.logp_p[tc];
      lq[k] = a.logp_q[tc];
    }
#pragma unroll
    for (int k = 0; k < kSeqUnroll; ++k)
      if (ok[k]) acc += (double)lp[k] - (double)lq[k];
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
  if constexpr (NW > 1) {
    __shared__ double sh[NW];
    if ((lane & 63) == 0) sh[lane >> 6] = acc;
    __syncthreads();
    acc = 0.0;
    for (int w = 0; w < NW; ++w) acc += sh[w];
  }
  if (lane == 0) a.logK[u] = acc;
}

// Response holding token t: the largest s in [lo, hi) with offsets[s] <= t, if t <
// offsets[s + 1]; -1 when no response holds t. Reads offsets[lo .. hi] only, whatever they hold.
// UNIFORM: t is the same for the whole workgroup, so the search takes scalar loads.
template <bool UNIFORM>
__device__ __forceinline__ int64_t find_response(const int64_t* off, int64_t lo, int64_t hi,
                                                 int64_t t) {
  auto at = [&](int64_t s) { return UNIFORM ? sload(off + s) : off[s]; };
  if (hi - lo < 1 || at(lo) > t) return -1;
  while (hi - lo > 1) {
    const int64_t mid = lo + (hi - lo) / 2;
    if (at(mid) <= t)
      lo = mid;
    else
      hi = mid;
  }
  return t < at(lo + 1) ? lo : -1;
}

// A sequence operator's weight of response s, from the pieces of its log K.
__device__ __forceinline__ float seq_weight(const PrepassArgs& a, int64_t s, bool& acted) {
  double lK = a.logK[s * a.pieces];
  for (int k = 1; k < a.pieces; ++k) lK += a.logK[s * a.pieces + k];
  if (a.ops.op == CIS_OP_SEQ_TIS) {
    acted = lK > log((double)a.ops.hi);
    return acted ? a.ops.hi : (float)exp(lK);
  }
  const bool keep = lK >= log((double)a.ops.lo) && lK <= log((double)a.ops.hi);
  acted = !keep;
  return keep ? (float)exp(lK) : 0.f;
}

// ------------------------------------------------------------------------------------------
// Per-token weights of an operator from recorded log-probabilities: w, acted, the
// displacement and the diagnostics (log k, k - w). The decoupled path runs it before the row
// kernel with l_p = l_old; cis_weights_ex runs it on its own. A workgroup takes 256 consecutive
// tokens at a time: the responses of the first and the last bound the tokens' searches, and
// where they are no more than the threads, each response's weight (float64 logarithms and
// exponential) is formed once and read from LDS. cis_weights_ex's statistics are summed here too
// (written per token and read again by one workgroup they took 98 us for 524288 tokens).
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kWeightsBlock) void cis_prepass_kernel(const PrepassArgs a) {
  __shared__ float sh_w[kWeightsBlock];
  __shared__ bool sh_acted[kWeightsBlock];
  if (a.queue && blockIdx.x == 0 && threadIdx.x < kRowQueues)
    a.queue[threadIdx.x * (kQueueStride / sizeof(*a.queue))] = 0ull;
  const bool seq = a.ops.op == CIS_OP_SEQ_TIS || a.ops.op == CIS_OP_SEQ_MIS;
  RowStats st{};
  for (int64_t t0 = (int64_t)blockIdx.x * kWeightsBlock; t0 < a.T;
       t0 += (int64_t)gridDim.x * kWeightsBlock) {
    const int64_t t = t0 + threadIdx.x;
    int64_t s_lo = 0, s_hi = a.n_seq;
    if (seq) {
      const int64_t tl = t0 + kWeightsBlock < a.T ? t0 + kWeightsBlock - 1 : a.T - 1;
      const int64_t x = find_response<true>(a.offsets, 0, a.n_seq, t0);
      if (x >= 0) s_lo = x;
      const int64_t y = x >= 0 && tl < sload(a.offsets + x + 1)
                            ? x
                            : find_response<true>(a.offsets, s_lo, a.n_seq, tl);
      if (y >= s_lo) s_hi = y + 1;
      __syncthreads();  // the previous tokens' weights have been read
      if (s_hi - s_lo <= kWeightsBlock && s_lo + threadIdx.x < s_hi)
        sh_w[threadIdx.x] = seq_weight(a, s_lo + threadIdx.x, sh_acted[threadIdx.x]);
      __syncthreads();
    }
    if (t >= a.T) continue;
    float w = 0.f, logk = 0.f, excess = 0.f, eps = 0.f;
    bool acted = false;
    const bool valid = token_valid(a.mask, a.ids, a.V, t);
    if (valid) {
      const float lp = a.logp_p[t], lq = a.logp_q[t];
      const float one_m_p = -expm1f(lp);
      logk = lp - lq;
      if (seq) {
        const int64_t s = find_response<false>(a.offsets, s_lo, s_hi, t);
        if (s >= 0 && s_hi - s_lo <= kWeightsBlock) {
          w = sh_w[s - s_lo];
          acted = sh_acted[s - s_lo];
        } else if (s >= 0) {
          w = seq_weight(a, s, acted);
        }
      } else {
        w = op_weight(a.ops, lp, lq, one_m_p, acted);
      }
      const float k = expf(logk);
      excess = (k == w) ? 0.f : k - w;
      eps = displacement(lp, lq, one_m_p);
    }
    if (a.w_out) a.w_out[t] = w;
    if (a.acted_out) a.acted_out[t] = acted ? 1 : 0;
    if (a.eps_out) a.eps_out[t] = eps;
    if (a.wpre_ws) a.wpre_ws[t] = w;
    if (a.pflags_ws) a.pflags_ws[t] = acted ? kFlagTrunc : 0;
    if (a.logk_ws) a.logk_ws[t] = logk;
    if (a.excess_ws) a.excess_ws[t] = excess;
    if (a.parts)
      take_row(st, 0.f, valid ? (uint8_t)(kFlagValid | (acted ? kFlagTrunc : 0)) : 0, logk, excess);
  }
  if (!a.parts) return;  // the loss path's statistics follow the rows
  st = block_stats<kWeightsBlock>(st);
  if (threadIdx.x == 0) a.parts[blockIdx.x] = st;
}

const void* seq_sum_kernel(int threads) {
  return threads == 64 ? (const void*)&cis_seq_sum_kernel<64>
                       : (const void*)&cis_seq_sum_kernel<kSeqBlock>;
}
const void* combine_kernel_ext(bool lane) {
  return lane ? (const void*)&cis_combine_lane_kernel<true> : (const void*)&cis_combine_kernel<true>;
}
const void* seg_grad_kernel_ext(int dtype) {
  return dtype == CIS_BF16 ? (const void*)&cis_seg_grad_kernel<Bf16, kSegGradBlock, kSegGradK, true>
                           : (const void*)&cis_seg_grad_kernel<F32, kSegGradBlock, kSegGradK, true>;
}
const void* prepass_kernel() { return (const void*)&cis_prepass_kernel; }

}  // namespace cis
