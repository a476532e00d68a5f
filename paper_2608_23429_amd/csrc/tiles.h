// How a launch's vectors are cut into the one-wave tiles of its blocks.  Plain
// index arithmetic, the same on the host and in the kernels.
#pragma once

#include <stdint.h>

#include <hip/hip_runtime_api.h>

namespace cheb {

// Tiles of R (one or two) runs of 64 vectors: a tile's runs lie 2^lg vectors
// from one another, R 2^lg vectors after R 2^lg vectors; what is left
// past the last whole R 2^lg is divided evenly.
constexpr uint32_t kRun = 64;
constexpr uint32_t kRunLg = 6;

struct RunTile {
  uint32_t first;   // first vector of its first run
  uint32_t stride;  // vectors from run to run
};

template <int R>
__host__ __device__ inline uint32_t run_tiles(uint32_t n_vec, uint32_t lg) {
  if (R == 1) return (n_vec + kRun - 1) / kRun;
  const uint32_t span = uint32_t(R) << lg, rest = n_vec & (span - 1);
  return n_vec / span * ((1u << lg) / kRun) + ((rest + R - 1) / R + kRun - 1) / kRun;
}

// Tile `tile` <= run_tiles<R>(n_vec, lg), n_vec < 2^31.  The one past the
// tiles is the block of a ragged tail.  Where the rest fills as many tiles as
// a whole span, that one lies in a span past n_vec (base > n_vec, by less than
// 2 kRun), so the rest is halved as a signed number: `even` is then 0.
template <int R>
__host__ __device__ inline RunTile run_tile(uint32_t tile, uint32_t n_vec, uint32_t lg) {
  if constexpr (R == 1) return {tile * kRun, 0};
  static_assert(R <= 2, "one or two runs");
  constexpr uint32_t kLgR = 1;
  const uint32_t whole = n_vec >> (lg + kLgR), span = tile >> (lg - kRunLg);
  const uint32_t base = span << (lg + kLgR);
  // The rest is shorter than a span, and so are its tiles: span == whole.
  const uint32_t half = uint32_t(int32_t(n_vec - base + 1u) >> 1);
  const uint32_t even = (half + kRun - 1) / kRun * kRun;
  return {base + (tile & ((1u << (lg - kRunLg)) - 1u)) * kRun, span < whole ? 1u << lg : even};
}

// Whether all runs of a tile of run_tile<R> end within n_vec.  Never so for
// the one past the tiles: its last run lies behind every vector, and its end,
// at most kRun past the last whole kRun, is far from wrapping.
template <int R>
__host__ __device__ inline bool whole_tile(const RunTile &t, uint32_t n_vec) {
  return t.first + uint32_t(R - 1) * t.stride + kRun <= n_vec;
}

}  // namespace cheb
