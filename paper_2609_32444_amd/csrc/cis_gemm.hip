// Dense products of the LM-head form (gfx950 MFMA): bf16 operands, row-major (K contiguous) or
// k-major in memory, float32 accumulation. Used for the logits of a row chunk (hidden * W^T, both
// row-major), the gradient with respect to the hidden states (G * W, W k-major) and the gradient
// of the head weight (G^T * hidden, both k-major); and G from stored logits.
//
// Tiling: a workgroup of 8 waves owns a 256 x 256 tile of C; each wave owns 128 x 64 as 8 x 4
// blocks of v_mfma_f32_16x16x32_bf16 (which sustains about 98% of the matrix cores' peak on this
// part against about 86% for the 32x32x16 form). K advances 64 at a time through two LDS slabs
// that the buffer unit fills directly (buffer loads that write LDS: no registers staged, no LDS
// store instructions). gemm_bf16_kernel says how the loads, the fragment reads and the MFMAs of
// consecutive slabs, and of consecutive tiles, overlap.
//
// LDS slab: 512 rows (A's 256, then B's) of 64 bf16 = 128 bytes, unpadded because one
// buffer->LDS instruction fills 1 KiB contiguously. The 16-byte chunk c of row r is stored at
// chunk c ^ (r & 7): a fragment read then touches 16 rows at one logical chunk without bank
// conflicts (measured with the LDS counters; without the swizzle every read is a 4-way
// conflict).
//
// MFMA operand layout (16x16x32): lane l supplies X[i = l % 16][k = 8 (l / 16) + j], j = 0..7,
// for both operands, and accumulator register r of lane l is the product's element
// (i = 4 (l / 16) + r, i' = l % 16) (checked on the device against an exact integer product).
// The B fragment is passed as the first operand, so a lane's four registers hold four
// consecutive columns of one row of C and the epilogue stores 16 bytes at a time.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "cis_gemm.h"

namespace cis {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) bf16x4* lds_bf16x4;
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kRsrcWord3 = 0x00020000;  // raw buffer, 32-bit data format

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, kRsrcWord3);
}

// Bytes of an R x K row-major matrix (row stride ld elements of 2 bytes) from row r0 on, K
// rounded up to whole 16-byte chunks (an aligned chunk that holds a valid element cannot cross
// into an unmapped page), clamped to kOobBase: the offsets of a tile's 256 rows stay below it
// (ld <= 2^22), and kOobBase plus any row offset lies beyond every resource. Rows past R lie
// beyond theirs. A load beyond its resource returns zeros.
__device__ __forceinline__ uint32_t span_bytes(int64_t R, int64_t r0, int64_t K, int64_t ld) {
  if (r0 >= R) return 0;
  const int64_t b = ((R - r0 - 1) * ld + (K + 7) / 8 * 8) * 2;
  return b > (int64_t)kOobBase ? kOobBase : (uint32_t)b;
}

// Logical work unit -> (split, tile). The smaller dimension's tiles run fastest, in groups of at
// most kTileGroup of them, then the larger dimension, then the next group: the 32 units in
// flight on an XCD form about 8 x 4 tiles and share their operand panels in its L2. Loads alone
// (no arithmetic, one slab ahead) of the 4096 x 151936 x 2048 product took 1.19 us per slab in
// groups of 8 against 1.33 us with all 16 row tiles fastest.
constexpr uint32_t kTileGroup = 8;
__device__ __forceinline__ void unit_tile(const GemmArgs& g, uint32_t lin, uint32_t& tm,
                                          uint32_t& tn, uint32_t& split) {
  const uint32_t mt = (uint32_t)((g.M + kGemmTile - 1) / kGemmTile);
  const uint32_t nt = (uint32_t)((g.N + kGemmTile - 1) / kGemmTile);
  split = lin / (mt * nt);
  uint32_t t = lin - split * (mt * nt);
  const uint32_t few = g.m_fastest ? mt : nt, many = g.m_fastest ? nt : mt;
  const uint32_t groups = (few + kTileGroup - 1) / kTileGroup;
  const uint32_t per = (few + groups - 1) / groups;   // tiles of the smaller dimension per group
  const uint32_t gi = t / (per * many);
  t -= gi * (per * many);
  const uint32_t h = few - gi * per < per ? few - gi * per : per;
  const uint32_t hi = t / h, lo = gi * per + (t - hi * h);
  tm = g.m_fastest ? lo : hi;
  tn = g.m_fastest ? hi : lo;
}

// Consecutive workgroup ids go to the 8 XCDs in turn and each XCD has an L2 of its own, so XCD
// x is given the contiguous run [xcd_first(x), xcd_first(x) + xcd_count(x)) of the n units.
__device__ __forceinline__ uint32_t xcd_count(uint32_t n, uint32_t x) {
  return n / kGemmQueues + (x < n % kGemmQueues ? 1 : 0);
}
__device__ __forceinline__ uint32_t xcd_first(uint32_t n, uint32_t x) {
  const uint32_t per = n / kGemmQueues, rem = n % kGemmQueues;
  return x < rem ? x * (per + 1) : rem * (per + 1) + (x - rem) * per;
}

// Work queues (thread 0 of a workgroup): the next unit of the home XCD's run, then of the other
// XCDs' runs in turn; -1 when all are taken, or without a queue. The first units of a run go to
// the workgroups of that XCD by their index (xcd_count(gridDim.x, x) of them); the counter hands
// out the others. `tried` counts the runs found empty (kept across calls), so a workgroup makes
// at most kGemmQueues failed attempts in all.
__device__ __forceinline__ int next_unit(const GemmArgs& g, uint32_t home, uint32_t& tried) {
  if (!g.queue) return -1;
  while (tried < (uint32_t)kGemmQueues) {
    const uint32_t x = (home + tried) % kGemmQueues;
    const uint32_t i = xcd_count(gridDim.x, x) + (uint32_t)atomicAdd(&g.queue[x], 1);
    if (i < xcd_count((uint32_t)g.units, x)) return (int)(xcd_first((uint32_t)g.units, x) + i);
    ++tried;
  }
  return -1;
}

// Two 16-byte buffer loads that write LDS: lane l stores at bytes lds + 16 l and lds + 8192 +
// 16 l (lds is the same for the whole wave). Counted by vmcnt. The voff are range-checked against
// the resource, soff is not. They are written in assembly, and have no register output, because
// the compiler puts a full vmcnt wait between such a load and a later LDS read that it cannot
// tell apart; the waits here are explicit and counted. (m0 needs one wait state before its use,
// and an SGPR that a vector instruction wrote five, which the compiler does not insert ahead of
// assembly; it sets m0 right before each use of its own.)
__device__ __forceinline__ void load_lds16x2(__amdgpu_buffer_rsrc_t r, uint32_t lds,
                                             uint32_t voff0, uint32_t voff1, uint32_t soff) {
  asm volatile(
      "s_mov_b32 m0, %0\n\ts_nop 3\n\tbuffer_load_dwordx4 %2, %4, %5 offen lds\n\t"
      "s_mov_b32 m0, %1\n\ts_nop 0\n\tbuffer_load_dwordx4 %3, %4, %5 offen lds"
      ::"s"(lds), "s"(lds + 8192), "v"(voff0), "v"(voff1), "s"(r), "s"(soff)
      : "memory");
}

// Workgroup barrier once this wave's LDS reads have landed and at most N of its vector-memory
// operations are outstanding. __syncthreads() would wait for every load in flight. The memory
// clobber keeps the compiler from moving LDS accesses across it.
template <int N>
__device__ __forceinline__ void wait_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

constexpr int kWaves = (kGemmTile / kGemmWaveM) * (kGemmTile / kGemmWaveN);  // 8
constexpr int kThreads = kWaves * 64;
constexpr int kTm = kGemmWaveM / 16, kTn = kGemmWaveN / 16;                 // 8 x 4 blocks
constexpr int kPieceBytes = kGemmTile / 2 * kGemmBK * 2;  // half of an operand's rows of a slab
constexpr int kOpBytes = 4 * kPieceBytes;                 // an operand's rows, both slabs
constexpr int kPieceLoads = kPieceBytes / (kThreads * 16);  // loads per wave and piece: 2
constexpr int kGroupLoads = 2 * kPieceLoads;             // two pieces are requested together
static_assert(kGemmBK == 64 && kWaves == 8 && kTm == 8 && kTn == 4 && kPieceLoads == 2,
              "the piece maps below");

// Epilogue of a tile: lane holds C[m][n .. n + 3] for m = m-block row + lane % 16,
// n = n-block column + 4 (lane / 16); 16-byte stores where the row allows them.
template <bool BETA>
__device__ __forceinline__ void store_tile(const GemmArgs& g, const f32x4 (&acc)[kTm][kTn],
                                           int64_t m0, int64_t n0, int64_t split) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave / (kGemmTile / kGemmWaveN), wn = wave % (kGemmTile / kGemmWaveN);
  const int fr = lane & 15, fq = lane >> 4;
  float* Cp = g.C + split * g.c_split_stride;
  const bool vec = g.c_vec;
#pragma unroll
  for (int i = 0; i < kTm; ++i) {
    const int64_t m = m0 + wm * kGemmWaveM + i * 16 + fr;
    if (m >= g.M) continue;
    float* crow = Cp + m * g.ldc;
#pragma unroll
    for (int j = 0; j < kTn; ++j) {
      const int64_t n = n0 + wn * kGemmWaveN + j * 16 + 4 * fq;
      f32x4 v = acc[i][j];
      if (vec && n + 3 < g.N) {
        if (BETA) v += *(const f32x4*)(crow + n);
        *(f32x4*)(crow + n) = v;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (n + e < g.N) crow[n + e] = BETA ? v[e] + crow[n + e] : v[e];
      }
    }
  }
}

constexpr float kLog2e = 1.44269504088896340736f;
constexpr float kMinRef = -0x1p127f;  // floor of a running max: keeps max * log2(e) finite

// Row-loss epilogue kEpiLse of a logits tile (rows m0.., vocabulary columns n0.., tile column
// tn): per row and wave, the max over the wave's 64 columns and the sum of exp(z - max) leaving
// out the sampled column, one pair in part[row * ldp + 4 tn + wn] (the four lanes of a row in a
// wave combine by shuffles; the combine kernel folds a row's pairs in this order). The lane
// holding the sampled column stores its logit in zy[row].
template <bool FULL>
__device__ __forceinline__ void lse_tile(const GemmArgs& g, const f32x4 (&acc)[kTm][kTn],
                                         int64_t m0, int64_t n0, int64_t tn,
                                         const int (&ep_y)[kGemmTile]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave / (kGemmTile / kGemmWaveN), wn = wave % (kGemmTile / kGemmWaveN);
  const int fr = lane & 15, fq = lane >> 4;
  const int N = (int)g.N;                                   // V <= 2^22
  const int nb = (int)n0 + wn * kGemmWaveN + 4 * fq;         // this lane's first column
  const int64_t pidx = tn * (kGemmTile / kGemmWaveN) + wn;
#pragma unroll
  for (int i = 0; i < kTm; ++i) {
    const int64_t m = m0 + wm * kGemmWaveM + i * 16 + fr;
    const bool row_ok = m < g.M;
    const int y = ep_y[wm * kGemmWaveM + i * 16 + fr];
    float mx = kMinRef;
#pragma unroll
    for (int j = 0; j < kTn; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (FULL || nb + j * 16 + e < N) mx = fmaxf(mx, acc[i][j][e]);
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float mb = mx * kLog2e;
    const int dy = y - nb;  // the sampled column in this lane's 4 x 4 columns?
    const bool has_y = dy >= 0 && dy < kTn * 16 && (dy & 15) < 4;
    float sm = 0.f;
    if (has_y) {  // the one lane of the row that holds y leaves it out element by element
#pragma unroll
      for (int j = 0; j < kTn; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int n = nb + j * 16 + e;
          const float x = __builtin_amdgcn_exp2f(__builtin_fmaf(acc[i][j][e], kLog2e, -mb));
          sm += ((FULL || n < N) && n != y) ? x : 0.f;
        }
    } else {
#pragma unroll
      for (int j = 0; j < kTn; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float x = __builtin_amdgcn_exp2f(__builtin_fmaf(acc[i][j][e], kLog2e, -mb));
          sm += (FULL || nb + j * 16 + e < N) ? x : 0.f;
        }
    }
    sm += __shfl_xor(sm, 16, 64);
    sm += __shfl_xor(sm, 32, 64);
    if (row_ok && has_y) {
#pragma unroll
      for (int j = 0; j < kTn; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (dy == j * 16 + e) g.e.zy[m] = acc[i][j][e];
    }
    if (row_ok && fq == 0) g.e.part[m * g.e.ldp + pidx] = float2{mx, sm};
  }
}

// dL/dz of logit z in column n of a row with parameters p: -coef exp(z - lse), evaluated as
// +-exp2(z log2(e) - b2), and coef (1 - p) at the sampled column; 0 for a row without gradient.
__device__ __forceinline__ float grad_value(const GradParams& p, float z, int64_t n) {
  const float x = __builtin_amdgcn_exp2f(__builtin_fmaf(z, kLog2e, -p.b2));
  return p.y < 0 ? 0.f : ((n == p.y) ? p.gy : (p.neg ? -x : x));
}

// Row-loss epilogue kEpiGrad: grad_value of every logit of the tile, rounded to bf16 (nearest
// even) into G.
__device__ __forceinline__ void grad_tile(const GemmArgs& g, const f32x4 (&acc)[kTm][kTn],
                                          int64_t m0, int64_t n0,
                                          const GradParams (&gp)[kGemmTile]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave / (kGemmTile / kGemmWaveN), wn = wave % (kGemmTile / kGemmWaveN);
  const int fr = lane & 15, fq = lane >> 4;
#pragma unroll
  for (int i = 0; i < kTm; ++i) {
    const int64_t m = m0 + wm * kGemmWaveM + i * 16 + fr;
    if (m >= g.M) continue;
    const GradParams p = gp[wm * kGemmWaveM + i * 16 + fr];
    __bf16* grow = g.e.G + m * g.e.ldg;
#pragma unroll
    for (int j = 0; j < kTn; ++j) {
      const int64_t n = n0 + wn * kGemmWaveN + j * 16 + 4 * fq;
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = grad_value(p, acc[i][j][e], n + e);
      const bf16x4 o = {(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
      if (n + 3 < g.N) {
        *(bf16x4*)(grow + n) = o;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (n + e < g.N) grow[n + e] = o[e];
      }
    }
  }
}

// What the epilogue needs of a tile's rows, in LDS before the tile's contraction ends (loading
// it in the epilogue would put a load latency after every tile).
template <int EPI>
struct EpiRows {
  int y[kGemmTile];            // kEpiLse, kEpiLseStore: sampled id, or -1 when outside [0, N)
};
template <>
struct EpiRows<kEpiGrad> {
  GradParams gp[kGemmTile];
};
template <>
struct EpiRows<kEpiStore> {};

// The operands of one unit, and its contraction range: of a row-major operand a resource at its
// tile's first row, of a k-major one the address of its tile's first column.
struct UnitSrc {
  __amdgpu_buffer_rsrc_t a, b;
  const __bf16 *pa, *pb;
  uint32_t m0, n0, split;
  int kbeg, kend;
};
template <bool KMA, bool KMB>
__device__ __forceinline__ UnitSrc unit_src(const GemmArgs& g, int u) {
  UnitSrc s;
  uint32_t tm = 0, tn = 0;
  s.split = 0;
  if (u >= 0) unit_tile(g, (uint32_t)u, tm, tn, s.split);
  s.m0 = tm * kGemmTile;
  s.n0 = tn * kGemmTile;
  s.kbeg = (int)(s.split * g.k_split);
  // (u < 0: nothing to contract and empty resources, so that the loads ahead of the last tile
  // read nothing)
  s.kend = u < 0 ? s.kbeg : (int)(s.kbeg + g.k_split < g.K ? s.kbeg + g.k_split : g.K);
  const __bf16 *A = static_cast<const __bf16*>(g.A), *B = static_cast<const __bf16*>(g.B);
  s.pa = A + s.m0;
  s.pb = B + s.n0;
  if (!KMA)
    s.a = make_rsrc(A + (int64_t)s.m0 * g.lda, u < 0 ? 0 : span_bytes(g.M, s.m0, g.K, g.lda));
  if (!KMB)
    s.b = make_rsrc(B + (int64_t)s.n0 * g.ldb, u < 0 ? 0 : span_bytes(g.N, s.n0, g.K, g.ldb));
  return s;
}

// A k-major operand's resource starts at row k of the contraction and ends with its last one
// (slab_bytes), so rows at or past the end read as zero, and nothing past the matrix is read;
// columns past the matrix are read where they lie within it (they reach only results that are not
// stored). (Formed right before an operand's loads, with 32-bit arithmetic where it can be: scalar
// instructions ahead of the first phase held both waves of a SIMD up, 8% of the product.)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t slab_rsrc(const __bf16* p, uint32_t cols,
                                                            uint32_t ld, uint32_t k, int left) {
  return make_rsrc((const char*)p + (uint64_t)k * (uint64_t)(ld * 2), slab_bytes(cols, ld, left));
}

// The products. A workgroup works through units (tiles, or a tile's share of a split
// contraction): its own first one, then with a queue further ones until all are taken.
//
// A slab of LDS is four pieces of 16 KiB: A0, A1 (per wave row the first and second 64 of its
// 128 tile rows) and B0, B1 (per wave column the first and second 32 of its 64 columns). A wave
// multiplies a slab in four phases of 16 MFMAs, one per pair of pieces, in an order that swaps
// the parts of B0 and B1 from slab to slab:
//
//   even slab (buffer 0):  A0 B0 | A0 B1 || A1 B1 | A1 B0 ||
//   odd slab  (buffer 1):  A0 B1 | A0 B0 || A1 B0 | A1 B1 ||
//
// so the fragments of a phase are always read from LDS one phase or more ahead, into registers
// whose last use has passed (A0, A1: 32 registers each, B0, B1: 16 each), and no MFMA waits for
// a read issued after a barrier. A barrier (||) every two phases frees two pieces, which are
// requested for the slab two ahead at once; they are waited for three such requests later (six
// phases, 1.5 slabs), and the two newer requests stay in flight (vmcnt(2 * kGroupLoads)). Loads
// alone, one slab ahead, take 1.2-1.5 us per slab here, and 0.92-1.16 us two slabs ahead.
// The same stream runs on into the next tile: its first two slabs are requested during the last
// two of this one, so the epilogue runs with them in flight. (Past the last unit, and past the
// end of the contraction, the loads are out of range and return zeros.) With an odd number of
// slabs the last odd slab's phases are left out and its pieces requested at once: 4096 x 151936 x
// 192 430 us when they multiplied zeros, 389 so; x 576 759 and 702, x 1600 1591 and 1536.
//
// What bounds it: the card's power, and the epilogue. With operands of zeros the same loop runs at
// 2.36 GHz and 2110-2230 TFLOP/s (2290-2390 clocks per slab, 2048 of them MFMAs); with random
// operands and no epilogue, one after another, the clock falls to 1.67-1.71 GHz (1423-1535
// TFLOP/s, the MFMAs busy for more than 80% of the clocks). Within a call the MFMAs are busy for less
// (counters, a pass of its own: 66% for dL/dh, 71% for dL/dW, 50% for the logits with their store,
// whose waves all store with no MFMAs to do), and the clock is higher for it: 2.04, 1.87 and 2.12 GHz.
// Products of the rollout batch, before (one slab ahead, every fragment read behind the slab's barrier) and now:
// logits with pairs, 4096 x 151936 x 2048, 2.07 and 1.84 ms; with the stored chunk 2.65 and
// 2.38 ms; dL/dh, 4096 x 2048 x 151936, 1.97 and 1.79 ms (1.68 with a transposed copy of W, which
// takes 0.22 ms per call); dL/dW, 151936 x 2048 x 16384, 8.62 and 7.39 ms (7.30 with transposed
// copies of G and h, for which a chunk's G and G^T took 1.03 ms instead of 0.65 ms for G).
//
// KMA, KMB: the operand is k-major in memory, [K, M] or [K, N], so a product needs no transposed
// copy. Its piece of a slab is 64 rows of 128 columns (256 bytes) in LDS, and a fragment is read
// by two transposing reads (ds_read_b64_tr_b16: within 16 lanes, lane 4a + b receives element b
// of the 8 bytes of lanes a, 4 + a, 8 + a and 12 + a). The 32-byte block c of row k is stored at
// block c ^ (k & 3 | (k >> 3 & 1) << 2): the eight rows that half a wave reads at once lie in
// different banks.
template <bool BETA, int EPI, bool KMA, bool KMB>
__global__ __launch_bounds__(kThreads) void gemm_bf16_kernel(const GemmArgs g) {
  // A's pieces (slab 0: A0, A1, slab 1: A0, A1), then B's: every fragment of an operand lies
  // within the 16-bit offset of one address
  __shared__ __attribute__((aligned(1024))) char lds[2 * kOpBytes];
  __shared__ EpiRows<EPI> er[2];   // of this unit and of the next
  __shared__ int sh_unit[2];       // the unit after this one
  constexpr bool kLse = EPI == kEpiLse || EPI == kEpiLseStore;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / (kGemmTile / kGemmWaveN), wn = wave % (kGemmTile / kGemmWaveN);
  const uint32_t lds0 =
      (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds + wave * 1024;

  const uint32_t home = blockIdx.x % kGemmQueues;
  uint32_t tried = 0;
  int u = (int)(xcd_first((uint32_t)g.units, home) + blockIdx.x / kGemmQueues);

  // Load j (0, 1) of a piece fills the 16-byte units (8 j + wave) 64 + lane of its 128 slab rows:
  // slab row 64 j + 8 wave + lane / 8, stored chunk lane % 8, holding logical chunk (lane % 8) ^
  // (row & 7). Slab rows to tile rows: a piece holds, per wave row (column) of the tile, 64 (32)
  // of its rows (columns), so that a wave's tile stays contiguous: piece h's row 64 j + x of A is
  // tile row 128 j + 64 h + x, row 32 c + x of B tile row 64 c + 32 h + x.
  // k-major: load j fills rows 32 j + 4 wave + lane / 16, stored chunk lane % 16 (half of a
  // 32-byte block) holding the logical block (lane % 16 / 2) ^ the row's swizzle.
  const int lchunk8 = ((lane & 7) ^ ((lane >> 3) & 7)) * 8;
  const int kcol = (((lane & 15) >> 1) ^ ((lane >> 4) | (((wave >> 1) & 1) << 2))) * 16 +
                   (lane & 1) * 8;   // column within a k-major piece
  const uint32_t va =
      KMA ? (uint32_t)(((wave * 4 + (lane >> 4)) * g.lda + kcol / 64 * 128 + kcol % 64) * 2)
          : (uint32_t)(((wave * 8 + (lane >> 3)) * g.lda + lchunk8) * 2);
  const uint32_t vb =
      KMB ? (uint32_t)(((wave * 4 + (lane >> 4)) * g.ldb + kcol / 32 * 64 + kcol % 32) * 2)
          : (uint32_t)(((wave / 4 * 64 + wave % 4 * 8 + (lane >> 3)) * g.ldb + lchunk8) * 2);
  // the resource of operand op (0: A, 1: B) for unit s's slab at k
  auto rsrc = [&](int op, const UnitSrc& s, int k) {
    if (op ? KMB : KMA)
      return op ? slab_rsrc(s.pb, (uint32_t)(g.N - s.n0), (uint32_t)g.ldb, k, s.kend - k)
                : slab_rsrc(s.pa, (uint32_t)(g.M - s.m0), (uint32_t)g.lda, k, s.kend - k);
    return op ? s.b : s.a;
  };
  // operand op, piece h, of the slab at k of a contraction up to kend, into buffer b, through
  // resource r. Chunks at or past kend read as zero; one of a row-major operand that straddles it
  // is cleared by fix().
  auto load = [&](int op, int h, int b, __amdgpu_buffer_rsrc_t r, int k, int kend) {
    const bool km = op ? KMB : KMA;
    const uint32_t ld2 = (uint32_t)((op ? g.ldb : g.lda) * 2);
    const uint32_t lds = lds0 + op * kOpBytes + (2 * b + h) * kPieceBytes;
    if (km) {
      const uint32_t v = (op ? vb : va) + h * (op ? 64 : 128);
      load_lds16x2(r, lds, v, v + 32 * ld2, 0);
    } else {
      const uint32_t step = (op ? 32 : 64) * ld2;
      const uint32_t v = (lchunk8 < kend - k ? (op ? vb : va) : kOobBase) + h * step;
      load_lds16x2(r, lds, v, v + (op ? 4 : 2) * step, (uint32_t)(k * 2));
    }
  };
  // Fragment addresses. Row-major: lane holds row 16 i + lane % 16 of its piece, logical chunk
  // 4 s + lane / 16; a block's first row is a multiple of 16, so the swizzle is lane & 7.
  // k-major: lane 4 r + a of a group g of 16 reads row 8 g + r (then 8 g + 4 + r) of step s,
  // columns 4 a .. 4 a + 3 of block i, and holds column lane % 16 with k = 8 g ... 8 g + 7.
  const int fr = lane & 15, fq = lane >> 4, sw = lane & 7;
  const int kr = fr >> 2, ksw = kr | ((fq & 1) << 2);
  const char* fa[KMA ? kTm / 2 : 2];
  const char* fb[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int c = ((4 * s + fq) ^ sw) * 16;
    if (!KMA) fa[s] = lds + (wm * 64 + fr) * 128 + c;
    if (!KMB) fb[s] = lds + kOpBytes + (wn * 32 + fr) * 128 + c;
  }
  const char* krow = lds + (8 * fq + kr) * 256 + (lane & 3) * 8;
  if constexpr (KMA) {
#pragma unroll
    for (int i = 0; i < kTm / 2; ++i) fa[i] = krow + ((wm * 4 + i) ^ ksw) * 32;
  }
  if constexpr (KMB) {
#pragma unroll
    for (int i = 0; i < kTn / 2; ++i) fb[i] = krow + kOpBytes + ((wn * 2 + i) ^ ksw) * 32;
  }
  auto read_tr = [&](const char* p) {
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4)p);
    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4)(p + 4 * 256));
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  };
  bf16x8 a0[kTm / 2][2], a1[kTm / 2][2], b0[kTn / 2][2], b1[kTn / 2][2];
  auto read_a = [&](bf16x8(&f)[kTm / 2][2], int h, int b, int q) {
    const int i = q % 4, s = q / 4, o = (2 * b + h) * kPieceBytes;
    if constexpr (KMA)
      f[i][s] = read_tr(fa[i] + o + s * 32 * 256);
    else
      f[i][s] = *(const bf16x8*)(fa[s] + o + i * 2048);
  };
  auto read_b = [&](bf16x8(&f)[kTn / 2][2], int h, int b, int q) {
    const int i = q % 2, s = q / 2, o = (2 * b + h) * kPieceBytes;
    if constexpr (KMB)
      f[i][s] = read_tr(fb[i] + o + s * 32 * 256);
    else
      f[i][s] = *(const bf16x8*)(fb[s] + o + i * 2048);
  };
  f32x4 acc[kTm][kTn];
  // One phase: the MFMAs of an A piece with a B piece, a fragment read (q = 0..7, if any) ahead of
  // each group of two, the loads of a piece ahead of the last; the fences keep that order.
  auto phase = [&](int ha, int hb, const bf16x8(&xa)[kTm / 2][2], const bf16x8(&xb)[kTn / 2][2],
                   auto read, auto loads) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int s = q / 4, i = q % 4;
      read(q);
      if (q == 7) loads();
#pragma unroll
      for (int j = 0; j < kTn / 2; ++j)
        acc[ha * 4 + i][hb * 2 + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
            xb[j][s], xa[i][s], acc[ha * 4 + i][hb * 2 + j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // Clears the elements at and past K of the slab in buffer b whose last chunk straddles K.
  // (Everything outstanding is waited for first: this is the last slab of a contraction whose
  // length is not a multiple of 8.)
  auto fix = [&](int b, int kend) {
    wait_barrier<0>();
    const int c = (kend % kGemmBK) / 8;
    char* p = lds + tid / 256 * kOpBytes + b * 2 * kPieceBytes + tid % 256 * 128 +
              ((c ^ (tid & 7)) * 16);   // a chunk of each of the slab's 512 rows
    bf16x8 e = *(const bf16x8*)p;
#pragma unroll
    for (int x = 0; x < 8; ++x)
      if (x >= kend % 8) e[x] = (__bf16)0.f;
    if (tid < 256 || !KMB) *(bf16x8*)p = e;   // (A's 256 rows, then B's)
    lds_barrier();
  };
  auto tail_slab = [](const UnitSrc& s) {   // the slab that fix() is for, or -1
    return !KMA && s.kend % 8 ? (s.kend - s.kbeg) / kGemmBK : -1;
  };
  // requests for the epilogue's inputs of unit s's rows, and their store to LDS
  auto epi_id = [&](const UnitSrc& s) -> int64_t {
    const int64_t m = (int64_t)s.m0 + tid;
    return kLse && tid < kGemmTile && m < g.M ? g.e.ids[m] : -1;
  };
  auto epi_gp = [&](const UnitSrc& s) -> GradParams {
    const int64_t m = (int64_t)s.m0 + tid;
    return EPI == kEpiGrad && tid < kGemmTile && m < g.M ? g.e.gp[m]
                                                         : GradParams{INFINITY, 0, 0.f, -1};
  };
  auto epi_put = [&](EpiRows<EPI>& r, int64_t y, const GradParams& p) {
    if (tid < kGemmTile) {
      if constexpr (kLse) r.y[tid] = (y >= 0 && y < g.N) ? (int)y : -1;
      if constexpr (EPI == kEpiGrad) r.gp[tid] = p;
    }
  };

  UnitSrc cur = unit_src<KMA, KMB>(g, u);
  // the first two slabs, in the order in which the stream requests pieces
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int k = cur.kbeg + b * kGemmBK;
    const __amdgpu_buffer_rsrc_t ra = rsrc(0, cur, k), rb = rsrc(1, cur, k);
    load(0, 0, b, ra, k, cur.kend);
    load(1, b, b, rb, k, cur.kend);
    load(1, 1 - b, b, rb, k, cur.kend);
    load(0, 1, b, ra, k, cur.kend);
  }
  epi_put(er[0], epi_id(cur), epi_gp(cur));
  if (tid == 0) sh_unit[0] = next_unit(g, home, tried);
  wait_barrier<0>();
  if (tail_slab(cur) == 0) fix(0, cur.kend);

  for (int p = 0;; p ^= 1) {
#pragma unroll
    for (int q = 0; q < 8; ++q) read_a(a0, 0, 0, q);
#pragma unroll
    for (int q = 0; q < 4; ++q) read_b(b0, 0, 0, q);
    const int un = __builtin_amdgcn_readfirstlane(sh_unit[p]);
    const UnitSrc nxt = unit_src<KMA, KMB>(g, un);
    lds_barrier();   // every wave has read A0 and B0
#pragma unroll
    for (int i = 0; i < kTm; ++i)
#pragma unroll
      for (int j = 0; j < kTn; ++j) acc[i][j] = f32x4{};
    const int tail = tail_slab(cur), tail_nxt = tail_slab(nxt);
    const int nk = cur.kend > cur.kbeg ? (cur.kend - cur.kbeg + 2 * kGemmBK - 1) / (2 * kGemmBK) * 2
                                       : 2;
    for (int kt = 0; kt < nk; kt += 2) {
      const bool last = kt + 2 >= nk;
      // the slabs two ahead: this unit's, or the next one's first two
      UnitSrc su = cur;
      if (last) su = nxt;
      const int k2 = last ? nxt.kbeg : cur.kbeg + (kt + 2) * kGemmBK, k3 = k2 + kGemmBK;
      __amdgpu_buffer_rsrc_t ra, rb;
      // even slab
      phase(0, 0, a0, b0, [&](int q) { if (q < 4) read_b(b1, 1, 0, q); },
            [&] { ra = rsrc(0, su, k2); load(0, 0, 0, ra, k2, su.kend); });
      phase(0, 1, a0, b1, [&](int q) { read_a(a1, 1, 0, q); },
            [&] { rb = rsrc(1, su, k2); load(1, 0, 0, rb, k2, su.kend); });
      if (kt + 1 == tail) fix(1, cur.kend);
      wait_barrier<2 * kGroupLoads>();
      phase(1, 1, a1, b1, [&](int q) { read_a(a0, 0, 1, q); },
            [&] { load(1, 1, 0, rb, k2, su.kend); });
      phase(1, 0, a1, b0, [&](int q) { if (q < 4) read_b(b1, 1, 1, q); },
            [&] { load(0, 1, 0, ra, k2, su.kend); });
      wait_barrier<2 * kGroupLoads>();
      if (cur.kend - cur.kbeg <= (kt + 1) * kGemmBK) {   // no odd slab: an odd number of them
        ra = rsrc(0, su, k3);
        rb = rsrc(1, su, k3);
        load(0, 0, 1, ra, k3, su.kend);
        load(1, 1, 1, rb, k3, su.kend);
        load(1, 0, 1, rb, k3, su.kend);
        load(0, 1, 1, ra, k3, su.kend);
        if (tail_nxt == 0) fix(0, su.kend);
        wait_barrier<2 * kGroupLoads>();
        break;
      }
      // odd slab
      phase(0, 1, a0, b1, [&](int q) { if (q < 4) read_b(b0, 0, 1, q); },
            [&] { ra = rsrc(0, su, k3); load(0, 0, 1, ra, k3, su.kend); });
      phase(0, 0, a0, b0, [&](int q) { read_a(a1, 1, 1, q); },
            [&] { rb = rsrc(1, su, k3); load(1, 1, 1, rb, k3, su.kend); });
      if (last ? tail_nxt == 0 : kt + 2 == tail) fix(0, su.kend);
      wait_barrier<2 * kGroupLoads>();
      phase(1, 0, a1, b0, [&](int q) { read_a(a0, 0, 0, q); },
            [&] { load(1, 0, 1, rb, k3, su.kend); });
      phase(1, 1, a1, b1, [&](int q) { if (q < 4) read_b(b0, 0, 0, q); },
            [&] { load(0, 1, 1, ra, k3, su.kend); });
      wait_barrier<2 * kGroupLoads>();
    }
    // The next unit's slab 0 is in LDS and its slab 1 on the way. Its epilogue inputs, and the
    // unit after it, are requested now and stored once this epilogue is through. (The fragments
    // that the last phases read of it are read again above: they would cost the epilogue 48
    // registers.)
    const int64_t y = epi_id(nxt);
    const GradParams gp = epi_gp(nxt);
    int u2 = -1;
    if (tid == 0 && un >= 0) u2 = next_unit(g, home, tried);
    if constexpr (kLse) {
      if ((int64_t)cur.n0 + kGemmTile <= g.N)
        lse_tile<true>(g, acc, cur.m0, cur.n0, cur.n0 / kGemmTile, er[p].y);
      else
        lse_tile<false>(g, acc, cur.m0, cur.n0, cur.n0 / kGemmTile, er[p].y);
    }
    if constexpr (EPI == kEpiGrad) grad_tile(g, acc, cur.m0, cur.n0, er[p].gp);
    if constexpr (EPI == kEpiStore || EPI == kEpiLseStore)
      store_tile<BETA>(g, acc, cur.m0, cur.n0, cur.split);
    if (un < 0) break;
    epi_put(er[p ^ 1], y, gp);
    if (tid == 0) sh_unit[p ^ 1] = u2;
    u = un;
    cur = nxt;
    lds_barrier();
  }
  // the (empty) loads ahead of the last unit must not outlive the workgroup's LDS
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// C = sum_s P[s]: the split-K partials summed in split order.
struct ReduceArgs {
  const float* P;
  float* C;
  int64_t M, N, ldc, split_stride;
  int32_t splits;
};

// Four elements per thread (VEC: rows of 16-byte vectors), the splits' loads independent.
template <bool VEC>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const ReduceArgs r) {
  constexpr int E = VEC ? 4 : 1;
  typedef float vec __attribute__((ext_vector_type(E)));
  const uint32_t per = (uint32_t)(r.N / E);   // vectors per row
  const int64_t total = r.M * per;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * 256) {
    const int64_t m = i / per;
    const int64_t n = (i - m * per) * E;
    vec s{};
#pragma unroll 4
    for (int k = 0; k < r.splits; ++k)
      s += *(const vec*)(r.P + k * r.split_stride + m * r.N + n);
    *(vec*)(r.C + m * r.ldc + n) = s;
  }
}

// G = the loss gradient of stored float32 logits, from each row's GradParams, in bf16 (the
// kEpiGrad formula): one row and 8 columns per thread. Bound by memory.
__global__ __launch_bounds__(kGradThreads) void grad_kernel(const GradArgs t) {
  const int64_t tiles = grad_tiles(t.V);
  const int64_t r = blockIdx.x / tiles;
  const int64_t c = (int64_t)(blockIdx.x - r * tiles) * kGradCols + threadIdx.x * 8;
  if (c >= t.V) return;
  const float* z = t.Z + r * t.ldz + c;
  __bf16* o = t.G + r * t.ldg + c;
  const GradParams gp = t.gp[r];
  if (c + 8 <= t.V) {
    const f32x4 x = __builtin_nontemporal_load((const f32x4*)z);
    const f32x4 y = __builtin_nontemporal_load((const f32x4*)z + 1);
    bf16x8 g;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      g[e] = (__bf16)grad_value(gp, x[e], c + e);
      g[4 + e] = (__bf16)grad_value(gp, y[e], c + 4 + e);
    }
    *(bf16x8*)o = g;
  } else {
    for (int e = 0; c + e < t.V; ++e) o[e] = (__bf16)grad_value(gp, z[e], c + e);
  }
}

constexpr int kPoolInts = GemmQueuePool::kSets * kGemmQueues;
__global__ __launch_bounds__(kPoolInts) void zero_queue_kernel(int* q) { q[threadIdx.x] = 0; }

int64_t gemm_tiles(const GemmArgs& g) {
  return ((g.M + kGemmTile - 1) / kGemmTile) * ((g.N + kGemmTile - 1) / kGemmTile);
}

// Launches `fn` over g.units units, one workgroup per CU at most (the LDS slabs allow one). With
// more units than CUs the workgroups take them from queues.
hipError_t launch_units(GemmArgs g, const void* fn, GemmQueuePool& queues, int num_cu,
                        hipStream_t stream) {
  g.queue = nullptr;
  if (g.units > num_cu) {
    if (hipError_t e = queues.take(&g.queue, stream)) return e;
  }
  const int64_t grid = g.queue ? num_cu : g.units;
  void* args[] = {&g};
  return hipLaunchKernel(fn, dim3((unsigned)grid), dim3(kThreads), args, 0, stream);
}

}  // namespace

// (A kernel rather than a memset node clears the counters, so that a call can be captured.)
hipError_t GemmQueuePool::take(int** queue, hipStream_t stream) {
  if (used == kSets) {
    void* zargs[] = {&base};
    if (hipError_t e = hipLaunchKernel((const void*)&zero_queue_kernel, dim3(1), dim3(kPoolInts),
                                       zargs, 0, stream))
      return e;
    used = 0;
  }
  *queue = base + kGemmQueues * used++;
  return hipSuccess;
}

hipError_t launch_gemm_epi(GemmArgs g, GemmQueuePool& queues, int num_cu, hipStream_t stream) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  g.m_fastest = g.M <= g.N;
  g.k_split = g.K > 0 ? g.K : 1;
  g.c_split_stride = 0;
  g.c_vec = g.epi == kEpiLseStore && ((uintptr_t)g.C % 16 == 0) && g.ldc % 4 == 0;
  g.units = gemm_tiles(g);
  const void* fn = g.epi == kEpiLse        ? (const void*)&gemm_bf16_kernel<false, kEpiLse, false, false>
                   : g.epi == kEpiGrad     ? (const void*)&gemm_bf16_kernel<false, kEpiGrad, false, false>
                   : g.epi == kEpiLseStore ? (const void*)&gemm_bf16_kernel<false, kEpiLseStore, false, false>
                                           : nullptr;
  if (!fn) return hipErrorInvalidValue;
  return launch_units(g, fn, queues, num_cu, stream);
}

// The number of splits with the shortest estimate: rounds of one unit per CU, each its share of
// the contraction and kUnitSlabs for its start and epilogue, and the reduction's traffic at
// 5 TB/s; in slabs of 1.35 us (measured of a full chip). A split keeps kMinSplitLen at least.
// 4096 x 2048 x 151936: 2 splits (1 unit per CU); 1777 x 1600 x 50257: 5 (245 units; 8 splits
// make 392, a second round half empty).
int64_t gemm_splitk_count(int64_t M, int64_t N, int64_t K, int64_t max_splits, int num_cu) {
  constexpr double kUnitSlabs = 6, kReduceSlabs = 4 / (5e12 * 1.35e-6);
  const int64_t tiles = ((M + kGemmTile - 1) / kGemmTile) * ((N + kGemmTile - 1) / kGemmTile);
  const double slabs = (double)K / kGemmBK;
  int64_t best = 1;
  double best_t = INFINITY;
  for (int64_t s = 1; s <= max_splits && (s == 1 || K >= s * kMinSplitLen); ++s) {
    const double rounds = (double)((tiles * s + num_cu - 1) / num_cu);
    const double t = rounds * (2 * ceil(slabs / (2 * s)) + kUnitSlabs) +
                     (s > 1 ? kReduceSlabs * (s + 1) * (double)M * (double)N : 0);
    if (t < best_t) best_t = t, best = s;
  }
  return best;
}

hipError_t launch_gemm_tn(GemmArgs g, bool beta, GemmQueuePool& queues, int num_cu,
                          hipStream_t stream) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  g.m_fastest = g.M <= g.N;
  g.k_split = g.K > 0 ? g.K : 1;
  g.c_split_stride = 0;
  g.c_vec = ((uintptr_t)g.C % 16 == 0) && g.ldc % 4 == 0;
  g.units = gemm_tiles(g);
  const void* fn = beta ? (const void*)&gemm_bf16_kernel<true, kEpiStore, true, true>
                        : (const void*)&gemm_bf16_kernel<false, kEpiStore, true, true>;
  return launch_units(g, fn, queues, num_cu, stream);
}

hipError_t launch_gemm_nn(GemmArgs g, float* partial, int64_t max_splits, GemmQueuePool& queues,
                          int num_cu, hipStream_t stream) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  const void* fn = (const void*)&gemm_bf16_kernel<false, kEpiStore, false, true>;
  // the smaller dimension's tiles run fastest
  g.m_fastest = g.M <= g.N;
  const int64_t splits = gemm_splitk_count(g.M, g.N, g.K, max_splits, num_cu);
  g.units = gemm_tiles(g) * splits;
  const bool c_aligned = ((uintptr_t)g.C % 16 == 0) && g.ldc % 4 == 0;
  if (splits <= 1) {
    g.k_split = g.K > 0 ? g.K : 1;
    g.c_split_stride = 0;
    g.c_vec = c_aligned;
    return launch_units(g, fn, queues, num_cu, stream);
  }
  // split-K: partial products into `partial` [splits][M][N], then summed in split order
  // (whole pairs of slabs, the unit of the loop)
  const int64_t kper =
      ((g.K + splits - 1) / splits + 2 * kGemmBK - 1) / (2 * kGemmBK) * (2 * kGemmBK);
  GemmArgs p = g;
  p.C = partial;
  p.ldc = g.N;
  p.k_split = kper;
  p.c_split_stride = g.M * g.N;
  p.c_vec = ((uintptr_t)partial % 16 == 0) && g.N % 4 == 0;
  if (hipError_t e = launch_units(p, fn, queues, num_cu, stream)) return e;
  ReduceArgs r{partial, g.C, g.M, g.N, g.ldc, g.M * g.N, (int32_t)splits};
  const bool vec = c_aligned && p.c_vec;
  const int64_t blocks = (g.M * g.N / (vec ? 4 : 1) + 255) / 256;
  const void* rfn = vec ? (const void*)&splitk_reduce_kernel<true>
                        : (const void*)&splitk_reduce_kernel<false>;
  void* args[] = {&r};
  return hipLaunchKernel(rfn, dim3((unsigned)(blocks < 4096 ? blocks : 4096)), dim3(256), args, 0,
                         stream);
}

hipError_t launch_grad(const GradArgs& t, hipStream_t stream) {
  GradArgs part = t;
  for (int64_t r0 = 0; r0 < t.rows; r0 += part.rows) {
    part.rows = grad_rows(t.rows - r0, t.V);
    part.Z = t.Z + r0 * t.ldz;
    part.G = t.G + r0 * t.ldg;
    part.gp = t.gp + r0;
    void* args[] = {&part};
    if (hipError_t e = hipLaunchKernel((const void*)&grad_kernel,
                                       dim3((unsigned)(grad_tiles(t.V) * part.rows)),
                                       dim3(kGradThreads), args, 0, stream))
      return e;
  }
  return hipSuccess;
}

}  // namespace cis
