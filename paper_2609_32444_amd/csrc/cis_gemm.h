// Internal interface of the LM-head products (cis_gemm.hip). Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "cis_internal.h"

namespace cis {

// Epilogues of the logits product z = h W^T of a row chunk (A = h, B = W):
//   kEpiLse:      per row and 64-column block (4 per 256-column tile tn), the pair (max, sum
//                 of exp(z - max) leaving out the sampled column) into
//                 part[row * ldp + 4 tn + wn], and the sampled logit into zy[row]; z itself
//                 is not stored;
//   kEpiGrad:     dL/dz of the row from its GradParams, rounded to bf16, into
//                 G[row * ldg + col];
//   kEpiLseStore: kEpiLse, and z into C (float32) as kEpiStore does.
enum { kEpiStore = 0, kEpiLse = 1, kEpiGrad = 2, kEpiLseStore = 3 };
struct GemmEpi {
  const int64_t* ids;       // [M] sampled ids (kEpiLse)
  float2* part;             // [M, ldp] (kEpiLse)
  float* zy;                // [M] (kEpiLse)
  int64_t ldp;
  const GradParams* gp;     // [M] (kEpiGrad)
  __bf16* G;                // [M, ldg] (kEpiGrad; ldg a multiple of 4)
  int64_t ldg;
};

// C[M, N] (float32, row stride ldc) = A * B (+ C when accumulating), or one of the row-loss
// epilogues above instead of C. A and B are bf16. For the epilogues A is [M, K] and B is [N, K],
// both row-major; launch_gemm_nn takes A as [M, K] and B as [K, N], launch_gemm_tn A as [K, M] and
// B as [K, N]. Row strides lda, ldb are multiples of 8 elements, at most 2^22, and bases 16-byte
// aligned; a matrix's rows are mapped up to a multiple of 8 elements. Any M, N, K >= 0. The fields
// after ldc are set by the launches.
struct GemmArgs {
  const void* A;
  const void* B;
  float* C;
  int64_t M, N, K, lda, ldb, ldc;
  bool m_fastest;           // tile order: M tiles fastest
  bool c_vec;               // C rows and base allow 16-byte stores
  int64_t k_split;          // contraction length per split
  int64_t c_split_stride;   // elements between the splits' partial outputs
  int64_t units;            // tiles x splits
  int* queue;               // kGemmQueues work counters (zero at launch), or null
  int epi;                  // kEpiStore, or a row-loss epilogue (set by the caller)
  GemmEpi e;
};

inline GemmArgs gemm_args(const void* A, const void* B, float* C, int64_t M, int64_t N,
                          int64_t K, int64_t lda, int64_t ldb, int64_t ldc) {
  GemmArgs g{};
  g.A = A;
  g.B = B;
  g.C = C;
  g.M = M;
  g.N = N;
  g.K = K;
  g.lda = lda;
  g.ldb = ldb;
  g.ldc = ldc;
  return g;
}

// G (bf16, row stride ldg) = the loss gradient of the logits Z (float32, row stride ldz), from
// each row's GradParams. Row strides are multiples of 8 elements and bases 16-byte aligned.
struct GradArgs {
  const float* Z;
  __bf16* G;
  const GradParams* gp;
  int64_t rows, V, ldz, ldg;
};

constexpr int kGemmWaveM = 128;     // C tile per wave: 128 rows x 64 columns (8 waves)
constexpr int kGemmWaveN = 64;
constexpr int kGemmQueues = 8;      // one work queue per XCD

// Device scratch for the products' work queues, one set of kGemmQueues counters per product. A
// kernel clears all the sets before the first is used and again when they are used up (one
// launch per kSets products rather than one each: about 5 us of every product's time).
struct GemmQueuePool {
  static constexpr int kSets = 8;
  int* base;                // kSets * kGemmQueues ints
  int used = kSets;
  hipError_t take(int** queue, hipStream_t stream);
};

// Number of K splits, up to max_splits, that launch_gemm_nn uses for an M x N x K product.
int64_t gemm_splitk_count(int64_t M, int64_t N, int64_t K, int64_t max_splits, int num_cu);

// Launches on `stream`. With more tiles than CUs, one workgroup per CU takes tiles from per-XCD
// queues until all are taken, so XCDs that run faster take over tiles of slower ones. Results do
// not depend on it: a tile is computed the same way by whichever workgroup takes it.
//
// A [M, K] * B [K, N] into C. Small products are split along K, up to max_splits, and the partials
// (`partial`: float32, max_splits * M * N elements, 16-byte aligned; unused with max_splits = 1)
// summed in a fixed order.
hipError_t launch_gemm_nn(GemmArgs g, float* partial, int64_t max_splits, GemmQueuePool& queues,
                          int num_cu, hipStream_t stream);
// A^T * B, A [K, M] and B [K, N]; `beta` adds the product to C instead of overwriting it.
hipError_t launch_gemm_tn(GemmArgs g, bool beta, GemmQueuePool& queues, int num_cu,
                          hipStream_t stream);
// The logits product of a row chunk with a row-loss epilogue (kEpiLse, kEpiGrad or
// kEpiLseStore; no split-K; C only with kEpiLseStore): M rows of h, N = V columns of W.
hipError_t launch_gemm_epi(GemmArgs g, GemmQueuePool& queues, int num_cu, hipStream_t stream);
hipError_t launch_grad(const GradArgs& t, hipStream_t stream);

}  // namespace cis
