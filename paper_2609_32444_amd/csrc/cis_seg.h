// Forward pass over long rows split into segments (the loss without the gradient): short-lived
// workgroups each reduce one segment of one row, a second kernel folds each row's partials.
//
//   * cis_seg_kernel: workgroup b takes segment b % nseg of row b / nseg (consecutive
//     workgroups read consecutive segments of a row). Each thread loads its K 16-byte vectors
//     at once, takes their max, then the exp-sum relative to that max with the sampled logit
//     left out; the workgroup combines its lanes (shuffles, then LDS in a fixed order) into one
//     (max, exp-sum) pair, stored in the workspace. The thread that holds the sampled logit
//     stores it. Invalid rows are not read. Workgroups go to the eight XCDs in turn, so with an
//     even number of segments the short last one would always fall to the same XCDs and leave
//     them idle early: the segments of a row are rotated by row >> rot (seg_rotation). 16384
//     rows of V = 64000 (8 segments) 374 us without and 331 with it (6.3 TB/s), V = 128256 (16)
//     711 and 653, V = 32000 (4) 196 and 186. The workgroups are short-lived: a persistent grid
//     whose workgroups walk segment after segment, with the next segment's loads in flight,
//     measured 10-30% slower.
//   * cis_combine_kernel: folds each row's partials in a fixed order, so the result does not
//     depend on which segment finished first, and runs the row kernel's epilogue. Rows of at
//     most kSegMax partials (every split row) take one lane each: the max of the partials, then
//     their rescaled sums in segment order, and the epilogue by that lane alone. Rows of more
//     partials (the LM head's 64-column pieces) take one wave each: lane l takes partials
//     l, l + 64, ..., then a fixed xor tree.
//
// A row's logits are read once, like the register-resident row kernel; the difference is the
// traffic pattern: many small independent reads per CU instead of one row-sized working set,
// which is what the read-only stream of this device favours.
#pragma once

#include "cis_row.h"
#include "cis_stats.h"

namespace cis {

// BLOCK threads take a segment of BLOCK * K vectors. RE: re-unpack the vectors for the
// exp-sum instead of keeping K * EPV floats alive from the max pass (fewer registers, one more
// VALU operation per logit). USE (compile-time: the test of a rotation at run time cost the plain
// order 2%): the segments in order, rotated, or for cis_seg_grad_kernel.
template <class E, int BLOCK, int K, bool RE, SegUse USE>
__global__ __launch_bounds__(BLOCK) void cis_seg_kernel(const RowArgs a, const SegArgs g) {
  constexpr int EPV = E::kPerVec;
  constexpr int NW = BLOCK / 64;
  constexpr int AUX = USE == SegUse::kGrad ? 0 : kAuxNT;
  __shared__ float sh_m[NW];
  __shared__ float sh_s[NW];
  const int V = a.V;
  const int64_t total = a.T * (int64_t)g.nseg;
  if (USE == SegUse::kGrad && blockIdx.x == 0 && threadIdx.x == 0) *g.done = 0u;
  for (int64_t b = blockIdx.x; b < total; b += gridDim.x) {
    int tid = threadIdx.x;
    const int64_t row = b / g.nseg;
    int seg = (int)(b - row * g.nseg);
    if (USE == SegUse::kRotated) {
      seg += (int)((uint32_t)(row >> g.rot) % (uint32_t)g.nseg);
      if (seg >= g.nseg) seg -= g.nseg;
    }
    const RowScalars rsc = fetch_row_scalars<false>(a, row);
    if (!rsc.valid(V)) continue;  // uniform: the whole workgroup skips the row
    const int y = (int)rsc.y;
    const __amdgpu_buffer_rsrc_t rs =
        make_rsrc((const char*)a.logits + row * a.row_bytes, (uint32_t)a.nvec * 16u);
    const int v0 = seg * g.segvec + tid;
    u32x4 r[K];
    static_for<K>([&](auto I) {
      constexpr int k = I;
      r[k] = bload_aux<AUX>(rs, (uint32_t)(v0 + k * BLOCK) * 16u);
    });
    // vectors that reach past the row (the ragged last one, and whole vectors beyond it in
    // the last segment) read as -inf
    const bool tail = (v0 + (K - 1) * BLOCK + 1) * EPV > V;
    float m = kMinRef;
    static_for<K>([&](auto I) {
      constexpr int k = I;
      float f[EPV];
      E::unpack(r[k], f);
      if (tail) mask_past_end<E>(f, v0 + k * BLOCK, V);
#pragma unroll
      for (int e = 0; e < EPV; ++e) m = fmaxf(m, f[e]);
    });
    if (RE) opaque(r);
    const float mb = m * kLog2e;
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    float zy_mine = 0.f;
    bool y_mine = false;
    const int vy = y / EPV;
    static_for<K>([&](auto I) {
      constexpr int k = I;
      float f[EPV];
      E::unpack(r[k], f);
      const int v = v0 + k * BLOCK;
      if (tail) mask_past_end<E>(f, v, V);
      if (v == vy) {  // one thread of one segment per row
        y_mine = true;
        accum_vec_skip<E>(f, mb, acc, true, y % EPV, zy_mine);
      } else {
        accum_vec<E>(f, mb, acc);
      }
    });
    float s = (acc[0] + acc[1]) + (acc[2] + acc[3]);
    wave_lse_reduce(m, s);
    if (y_mine) g.zy[row] = zy_mine;
    if (NW == 1) {
      if (tid == 0) g.part[row * g.stride + seg] = float2{m, s};
      continue;
    }
    const int wid = tid >> 6;
    if ((tid & 63) == 0) {
      sh_m[wid] = m;
      sh_s[wid] = s;
    }
    __syncthreads();
    if (tid == 0) {
      float M = sh_m[0], S = sh_s[0];
#pragma unroll
      for (int w = 1; w < NW; ++w) lse_combine(M, S, sh_m[w], sh_s[w]);
      g.part[row * g.stride + seg] = float2{M, S};
    }
    __syncthreads();  // sh_m / sh_s are reused by the next segment of this workgroup
  }
}

// The gradient of few long rows, after cis_seg_kernel (same segments): a workgroup folds its row's
// pairs, runs the row's epilogue (each wave redundantly; the first segment's workgroup stores the
// row's outputs) and writes its segment of the gradient. The workgroup whose row is the last to be
// stored sums the statistics: rows are counted in g.done, cleared by cis_seg_kernel.
// With fewer rows than compute units the row kernel leaves most of the chip idle and takes a
// row's whole latency (96 rows of V = 151936: 19.5 us of 20.8); the segments spread over all of
// it (8.7 and 10.4 us), and the second read of the logits comes from the caches: cis_seg_kernel
// reads them with the default policy for that (non-temporal: 19.6 against 17.9 us per call), and
// both kernels put a segment on the same XCD.
template <class E, int BLOCK, int K, bool EXT>
__global__ __launch_bounds__(BLOCK) void cis_seg_grad_kernel(const RowArgs a, const SegArgs g,
                                                             const FinalizeArgs fa) {
  constexpr int EPV = E::kPerVec;
  __shared__ bool sh_last;
  const int tid = threadIdx.x, lane = tid & 63;
  const int64_t row = blockIdx.x / g.nseg;
  const int seg = (int)(blockIdx.x - row * g.nseg);
  const RowScalars rsc = fetch_row_scalars<EXT>(a, row);
  const bool valid = rsc.valid(a.V), writer = seg == 0 && tid == 0;
  const bool ragged = a.V % EPV != 0;
  const __amdgpu_buffer_rsrc_t rs =
      make_rsrc((const char*)a.logits + row * a.row_bytes, valid ? (uint32_t)a.nvec * 16u : 0u);
  void* grow = (char*)a.dlogits + row * a.grow_bytes;
  const __amdgpu_buffer_rsrc_t ws = make_rsrc(grow, (uint32_t)(a.nvec - (ragged ? 1 : 0)) * 16u);
  const int v0 = seg * g.segvec + tid;
  u32x4 r[K];
  static_for<K>([&](auto I) { r[I] = bload(rs, (uint32_t)(v0 + I * BLOCK) * 16u, 0u); });
  float coef = 0.f, b2 = INFINITY, gy = 0.f;
  if (valid) {
    float m = kMinRef, s = 0.f;
    if (lane < g.nseg) {
      const float2 p = g.part[row * g.stride + lane];
      m = p.x;
      s = p.y;
    }
    wave_lse_reduce(m, s);
    const RowResult rr = row_epilogue<EXT, true>(a, rsc, row, m, s, g.zy[row], writer);
    coef = rr.coef;
    gy = coef * rr.one_m_p;
    if (coef != 0.f) b2 = (rr.lse - logf(fabsf(coef))) * kLog2e;
  } else if (writer) {
    row_invalid<EXT, true>(a, rsc, row);
  }
  const uint32_t sgn = coef > 0.f ? E::kSignMask : 0u;
  const int vy = valid ? (int)rsc.y / EPV : -1;
  static_for<K>([&](auto I) {
    const int v = v0 + I * BLOCK;
    const u32x4 out = valid ? grad_vec<E>(r[I], b2, sgn) : u32x4{0u, 0u, 0u, 0u};
    bstore(out, ws, (uint32_t)v * 16u, 0u);
    if (ragged && v == a.nvec - 1)
      for (int e = 0; e < a.V - (a.nvec - 1) * EPV; ++e)
        E::store_elem(grow, v * EPV + e, E::elem_bits(out, e));
    if (v == vy) E::store_elem(grow, (int)rsc.y, E::bits_of(gy));   // (after its own vector's)
  });
  if (seg != 0) return;
  if (tid == 0) sh_last = last_done(g.done, (uint32_t)a.T);
  __syncthreads();
  if (!sh_last) return;
  RowStats st{};
  for (int64_t t = tid; t < a.T; t += BLOCK)
    take_row(st, get_dev(fa.terms_ws + t), get_dev(fa.flags_ws + t), get_dev(fa.logk_ws + t),
             get_dev(fa.excess_ws + t));
  st = block_stats<BLOCK>(st);
  if (tid == 0) write_stats(fa, st);
}

// GradParams of a row for the fused LM-head pass: the row kernel's gradient
// -coef exp(z - lse) = s exp2(z log2(e) - b2), and coef (1 - p) at y.
__device__ __forceinline__ GradParams grad_params(const RowResult& rr, int64_t y) {
  const float coef = rr.coef;
  const float b2 = coef != 0.f ? (rr.lse - logf(fabsf(coef))) * kLog2e : INFINITY;
  return GradParams{b2, coef > 0.f ? 1 : 0, coef * rr.one_m_p, (int32_t)y};
}

template <bool EXT>
__global__ __launch_bounds__(kCombineBlock) void cis_combine_lane_kernel(const RowArgs a,
                                                                         const SegArgs g) {
  const int64_t row = (int64_t)blockIdx.x * kCombineBlock + threadIdx.x;
  if (row >= a.T) return;  // no barrier follows
  const RowScalars rsc = fetch_row_scalars_lane<EXT>(a, row);
  if (!rsc.valid(a.V)) {
    row_invalid<EXT>(a, rsc, row);
    if (g.gp) g.gp[row] = GradParams{INFINITY, 0, 0.f, -1};
    return;
  }
  const float2* pr = g.part + row * g.stride;
  float M = kMinRef;
  for (int k = 0; k < g.nseg; ++k) M = fmaxf(M, pr[k].x);
  float s = 0.f;
  for (int k = 0; k < g.nseg; ++k) {
    const float2 p = pr[k];
    s += p.y * fast_exp2((p.x - M) * kLog2e);
  }
  const RowResult rr = row_epilogue<EXT>(a, rsc, row, M, s, g.zy[row], true);
  if (g.gp) g.gp[row] = grad_params(rr, rsc.y);
}

template <bool EXT>
__global__ __launch_bounds__(kCombineBlock) void cis_combine_kernel(const RowArgs a,
                                                                    const SegArgs g) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * (kCombineBlock / 64) +
                      (__builtin_amdgcn_readfirstlane(threadIdx.x) >> 6);
  if (row >= a.T) return;  // whole waves leave together; no barrier follows
  const RowScalars rsc = fetch_row_scalars<EXT>(a, row);
  if (!rsc.valid(a.V)) {
    if (lane == 0) {
      row_invalid<EXT>(a, rsc, row);
      if (g.gp) g.gp[row] = GradParams{INFINITY, 0, 0.f, -1};
    }
    return;
  }
  float m = kMinRef, s = 0.f;
  for (int k = lane; k < g.nseg; k += 64) {
    const float2 p = g.part[row * g.stride + k];
    lse_combine(m, s, p.x, p.y);
  }
  wave_lse_reduce(m, s);
  const float zy = g.zy[row];
  const RowResult rr = row_epilogue<EXT>(a, rsc, row, m, s, zy, lane == 0);
  if (g.gp && lane == 0) g.gp[row] = grad_params(rr, rsc.y);
}

}  // namespace cis
