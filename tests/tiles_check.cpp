// The kernels' division of a launch into tiles, on the CPU: for vector counts
// over several spans and for the last ones a launch accepts, every vector
// belongs to exactly one run, no run of a whole tile ends past the end, and
// the block after the tiles, the ragged tail's, is never a whole tile.
#include <stdio.h>
#include <stdlib.h>

#include <algorithm>
#include <utility>
#include <vector>

#include "tiles.h"

using namespace cheb;

static void fail_at(const char *what, int runs, uint32_t n_vec, uint32_t block) {
  fprintf(stderr, "%s: %d runs, %u vectors, block %u\n", what, runs, n_vec, block);
  exit(1);
}

// Tiles from `from` on hold the vectors from `begin` on, each once.
template <int R>
static void check(uint32_t n_vec, uint32_t lg, uint32_t from, uint32_t begin) {
  const uint32_t n_tiles = run_tiles<R>(n_vec, lg);
  std::vector<std::pair<uint64_t, uint64_t>> runs;
  for (uint32_t b = from; b < n_tiles; ++b) {
    const RunTile t = run_tile<R>(b, n_vec, lg);
    for (uint32_t r = 0; r < uint32_t(R); ++r) {
      const uint64_t first = uint64_t(t.first) + uint64_t(r) * t.stride;
      uint64_t end = first + kRun;
      if (end > n_vec) {
        if (whole_tile<R>(t, n_vec)) fail_at("a whole tile ends past the end", R, n_vec, b);
        end = std::max(first, uint64_t(n_vec));
      }
      if (end > first) runs.emplace_back(first, end);
    }
  }
  std::sort(runs.begin(), runs.end());
  uint64_t at = begin;
  for (const auto &r : runs) {
    if (r.first != at) fail_at("a vector is left out or done twice", R, n_vec, from);
    at = r.second;
  }
  if (at != n_vec) fail_at("the last vectors are left out", R, n_vec, from);
  // The kernel tests for whole tiles first, so the tail's block must not be one.
  if (whole_tile<R>(run_tile<R>(n_tiles, n_vec, lg), n_vec))
    fail_at("the tail's block is taken for a tile", R, n_vec, n_tiles);
}

int main() {
  constexpr uint32_t kLg = 12, kSpan = 2u << kLg;  // the kernels' pairs of runs
  for (uint32_t n = 0; n <= 2 * kSpan + 130; ++n) {
    check<1>(n, kRunLg, 0, 0);
    check<2>(n, kLg, 0, 0);
  }
  // The last three spans below 2^31 vectors.
  const uint32_t end = 1u << 31, begin = end - 3 * kSpan;
  for (uint32_t n = end - kSpan - 300; n != end; ++n) {
    check<1>(n, kRunLg, begin / kRun, begin);
    check<2>(n, kLg, begin / kSpan * (kSpan / 2 / kRun), begin);
  }
  printf("tiles ok\n");
  return 0;
}
