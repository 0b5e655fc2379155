// Launch index -> output tile, shared by the matrix-core kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "repops_internal.h"

namespace repops {

// Map the launch-order tile index so that the tiles one XCD receives (the
// hardware deals workgroups round-robin over 8 XCDs) form a compact panel of
// GROUP_M tile rows, which share A and B slices in that XCD's L2.
__device__ __forceinline__ void tile_coords(int64_t t, int64_t ntiles, int64_t tiles_m,
                                            int64_t tiles_n, int64_t* bz, int64_t* tm,
                                            int64_t* tn) {
  constexpr int64_t kXcd = 8, kGroupM = 4;
  if (ntiles % kXcd == 0) t = (t % kXcd) * (ntiles / kXcd) + t / kXcd;
  const int64_t per_batch = tiles_m * tiles_n;
  *bz = t / per_batch;
  const int64_t r = t % per_batch;
  const int64_t group = r / (kGroupM * tiles_n);
  const int64_t first_m = group * kGroupM;
  const int64_t gsize = (tiles_m - first_m) < kGroupM ? (tiles_m - first_m) : kGroupM;
  const int64_t in_group = r % (kGroupM * tiles_n);
  *tm = first_m + in_group % gsize;
  *tn = in_group / gsize;
}

// Causal products (per batch element, row i, column j, contraction index kk).
// causal == 1: only outputs with j <= i are wanted, so a tile whose first
// column lies past its last row is skipped (its outputs are left unwritten).
// causal == 2: A is zero at kk > i, so a row tile starting at m0 needs k only
// up to the end of the k block holding row m0 + bm - 1's diagonal; every later
// block is a chain of zero products, whose partial is +0 and leaves acc
// unchanged (acc + (+0) = acc; acc is never -0), so skipping it keeps the bits.
__device__ __forceinline__ bool tile_above_diagonal(const GemmArgs& g, int64_t m0, int bm,
                                                    int64_t n0) {
  return g.causal == 1 && n0 > m0 + bm - 1;
}

__device__ __forceinline__ int64_t k_extent(const GemmArgs& g, int64_t m0, int bm) {
  if (g.causal != 2 || g.k_block <= 0) return g.k;
  const int64_t end = (m0 + bm + g.k_block - 1) / g.k_block * g.k_block;
  return end < g.k ? end : g.k;
}

// With causal == 1, square tiles and at least as many tile columns as rows,
// the launch covers only the tiles at or below each batch element's diagonal
// (tn <= tm): tile r of a batch element is the r-th of the lower triangle in
// row order.
__device__ __host__ __forceinline__ bool causal_triangle(int causal, int bm, int bn,
                                                         int64_t tiles_m, int64_t tiles_n) {
  return causal == 1 && bm == bn && tiles_n >= tiles_m;
}

// Tile of launch index t for any product: the lower triangle's tiles only (see
// causal_triangle), or every tile with tile_coords -- row tiles in reverse order
// when A is zero above its diagonal (causal == 2), so that the row tiles with
// the longest contraction start first.
__device__ __forceinline__ void tile_of(const GemmArgs& g, int bm, int bn, int64_t t,
                                        int64_t ntiles, int64_t tiles_m, int64_t tiles_n,
                                        int64_t* bz, int64_t* tm, int64_t* tn) {
  if (causal_triangle(g.causal, bm, bn, tiles_m, tiles_n)) {
    constexpr int64_t kXcd = 8;
    if (ntiles % kXcd == 0) t = (t % kXcd) * (ntiles / kXcd) + t / kXcd;
    const int64_t per = tiles_m * (tiles_m + 1) / 2;
    *bz = t / per;
    const int64_t r = t % per;
    // the last row tile whose triangle starts at or before r (integer
    // bisection; r < per, so it lies below tiles_m)
    int64_t row = 0, hi = tiles_m - 1;
    while (row < hi) {
      const int64_t mid = (row + hi + 1) / 2;
      if (mid * (mid + 1) / 2 <= r) row = mid; else hi = mid - 1;
    }
    *tm = row;
    *tn = r - row * (row + 1) / 2;
    return;
  }
  tile_coords(t, ntiles, tiles_m, tiles_n, bz, tm, tn);
  if (g.causal == 2) *tm = tiles_m - 1 - *tm;
}

}  // namespace repops
