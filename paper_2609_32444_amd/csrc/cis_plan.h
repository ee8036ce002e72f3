// Sizes and bounds that the launches and the kernels share: plain C++, so that a host program can
// check them over their whole range.
#pragma once

#include <stdint.h>

namespace cis {

constexpr int kGemmTile = 256;      // C tile per workgroup (rows and columns)
constexpr int kGemmBK = 64;         // contraction slab

// Bytes of a k-major operand from a slab's first element on that the slab's loads may touch: `left`
// rows of the contraction from there (its last one included), `cols` columns of the matrix from
// the tile's first one, row stride ld (a multiple of 8, at least cols rounded up to 8). A slab's
// loads cover kGemmBK rows of kGemmTile columns, in 16-byte chunks; those past the matrix's columns
// lie in its next rows, so a narrow matrix ends before the last of them does. With more rows than
// the loads reach (a row has at least 8 elements) they need no bound: kOobBase, beyond every offset
// of a tile. (All within 32 bits: ld <= 2^22.)
constexpr uint32_t kOobBase = 0x80000000u;
constexpr uint32_t slab_bytes(uint32_t cols, uint32_t ld, int left) {
  constexpr int reach = kGemmBK + kGemmTile / 8;
  const uint32_t last = ((uint32_t)(left - 1) * ld + ((cols + 7) & ~7u)) * 2;
  return left <= 0 ? 0u : left > reach ? kOobBase : last;
}

// grad_kernel: a workgroup of kGradThreads takes kGradCols columns of a row. Rows per launch: HIP
// refuses a launch of 2^32 work items, which 8192 rows of 2^22 columns reach.
constexpr int kGradThreads = 256;
constexpr int kGradCols = kGradThreads * 8;
constexpr int64_t kGradMaxBlocks = int64_t(1) << 20;
constexpr int64_t grad_tiles(int64_t V) { return (V + kGradCols - 1) / kGradCols; }
constexpr int64_t grad_rows(int64_t rows, int64_t V) {
  const int64_t most = kGradMaxBlocks / grad_tiles(V);   // V <= 2^22: at least 512
  return rows < most ? rows : most;
}

// Workgroups of kSeqBlock threads that sum a response's log K, or 0: a wave for each response. A
// wave up to kSeqWaveLen tokens on average (a workgroup would idle there), and with more responses
// than the work items of a launch allow workgroups of (HIP refuses 2^32; a wave each takes 64). With
// few long responses several workgroups for each, as far as their sums fit (`sums` of them in all) and
// have 2048 tokens each (two per thread).
constexpr int kSeqBlock = 1024;
constexpr int64_t kSeqWaveLen = 512;
constexpr int64_t kSeqMaxBlocks = int64_t(1) << 20;
constexpr int64_t seq_pieces(int64_t T, int64_t n_seq, int64_t sums) {
  const int64_t avg = T / n_seq;
  if (avg <= kSeqWaveLen || n_seq > kSeqMaxBlocks) return 0;
  const int64_t fit = sums / n_seq, work = avg / 2048;
  const int64_t pieces = fit < work ? fit : work;
  return pieces < 1 ? 1 : pieces;
}

}  // namespace cis
