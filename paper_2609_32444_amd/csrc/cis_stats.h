// Per-call statistics (cis_stats_t) summed over rows: a thread's share, a workgroup's sum in a
// fixed tree, and the results.
#pragma once

#include "cis_internal.h"

namespace cis {

__device__ __forceinline__ void take_row(RowStats& s, float term, uint8_t f, float lk, float ex) {
  s.loss += (double)term;
  s.valid += (f & kFlagValid) ? 1 : 0;
  s.bad_id += (f & kFlagBadId) ? 1 : 0;
  s.nonfinite += (f & kFlagNonFinite) ? 1 : 0;
  s.acted += (f & kFlagTrunc) ? 1 : 0;
  if (f & kFlagValid) {
    s.max_logk = fmaxf(s.max_logk, fabsf(lk));  // fmaxf ignores NaN
    s.excess += (double)ex;
  }
}

__device__ __forceinline__ void add_stats(RowStats& s, const RowStats& o) {
  s.loss += o.loss;
  s.excess += o.excess;
  s.max_logk = fmaxf(s.max_logk, o.max_logk);
  s.valid += o.valid;
  s.bad_id += o.bad_id;
  s.nonfinite += o.nonfinite;
  s.acted += o.acted;
}

// Sum over the workgroup's BLOCK threads, in thread 0.
template <int BLOCK>
__device__ __forceinline__ RowStats block_stats(RowStats s) {
  constexpr int NW = BLOCK / 64;
  __shared__ RowStats sh[NW];
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    RowStats o;
    o.loss = __shfl_down(s.loss, off, 64);
    o.excess = __shfl_down(s.excess, off, 64);
    o.max_logk = __shfl_down(s.max_logk, off, 64);
    o.valid = __shfl_down(s.valid, off, 64);
    o.bad_id = __shfl_down(s.bad_id, off, 64);
    o.nonfinite = __shfl_down(s.nonfinite, off, 64);
    o.acted = __shfl_down(s.acted, off, 64);
    add_stats(s, o);
  }
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0)
    for (int w = 1; w < NW; ++w) add_stats(s, sh[w]);
  return s;
}

// One thread of each of n participants calls this once its values are stored (device scope): true
// for the last of them. `done` starts at zero. (Returning atomics on one counter are served at about
// 80 M/s: for a few hundred participants.)
__device__ __forceinline__ bool last_done(uint32_t* done, uint32_t n) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the values are visible everywhere
  return __hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n - 1;
}

__device__ __forceinline__ void write_stats(const FinalizeArgs& a, const RowStats& s) {
  cis_stats_t r;
  r.loss = s.loss;
  r.n_valid = s.valid;
  r.n_bad_id = s.bad_id;
  r.n_nonfinite = s.nonfinite;
  r.n_trunc = s.acted;
  r.max_abs_logk = (double)s.max_logk;
  r.trunc_excess = s.excess;
  r.reserved = 0;
  *a.stats = r;
  if (a.stats_copy) *a.stats_copy = r;
  if (a.loss_out) *a.loss_out = (float)s.loss;
}

}  // namespace cis
