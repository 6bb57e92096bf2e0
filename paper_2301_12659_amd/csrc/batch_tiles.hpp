// The tiles that the batched assembly turns through LDS: tile_rows entries
// (i, j) of a path's Jacobian with all D coefficients, fewer rows at large orders.
// A launch holds paths of every order, and its LDS is the largest tile among
// them: the tiles do not grow with D (64 coefficients take more than 65).
#pragma once

namespace mdk {

__host__ __device__ inline int tile_rows(int D) { return D <= 64 ? 16 : 8; }

// Where limb l of coefficient s of a tile's row is, in doubles.
__host__ __device__ inline int tile_index(int D, int l, int s, int row) { return (l * D + s) * (tile_rows(D) + 1) + row; }

// Doubles per limb of a tile of order D; `most`: of the tiles so far.
__host__ __device__ inline int tile_doubles(int most, int D) {
  const int d = (tile_rows(D) + 1) * D;
  return d > most ? d : most;
}

}  // namespace mdk
