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
// lie in its next rows, so a narrow matrix ends before the last of them does. Rows further down
// than the loads reach (a row has at least 8 elements) need not be counted, which keeps the
// arithmetic within 32 bits (ld <= 2^22).
constexpr uint32_t slab_bytes(uint32_t cols, uint32_t ld, int left) {
  constexpr int reach = kGemmBK + kGemmTile / 8;
  const int rows = left < reach ? left : reach;
  return rows <= 0 ? 0u : ((uint32_t)(rows - 1) * ld + ((cols + 7) & ~7u)) * 2;
}

}  // namespace cis
