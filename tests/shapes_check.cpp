// The kernels' launch shapes, on the CPU.  Predictions: pairs of runs only where
// the library holds that kernel, and no pairs of interleaved entries, whose
// chunks they would leave.  Residuals: over every history size,
// storage type, layout and number of covering segments, and sizes up to the
// last one a residual may have, the grid stays within HIP's 2^32 - 1 threads.
// Reserved LDS lets as many blocks onto a compute unit as wanted and (to 12, where
// the unit it is handed out in still tells them apart) no more, and none is
// reserved where the caller wants it free.
#include <stdio.h>
#include <stdlib.h>

#include "shapes.h"
#include "tiles.h"

using namespace cheb;

static void check_grid(int ns, int vec, int ncover, uint32_t n_vec, bool contiguous) {
  const uint32_t singles = run_tiles<1>(n_vec, kRunLg);
  const ResShape s =
      within_grid(residual_shape(ns, vec, ncover, singles, contiguous, 256), singles);
  const uint64_t tiles = s.runs == 2 ? run_tiles<2>(n_vec, 12) : singles;
  const uint64_t per_block = uint64_t(s.waves) * uint64_t(s.tiles);
  const uint64_t threads = (tiles + s.tiles - 1) / s.tiles * 64u * per_block;
  // The kernels that are held: waves share a tile or have one each.
  const bool held = s.tiles == 1 ? s.waves == 1 || s.waves == 2 || s.waves == 4 ||
                                       (s.waves == 16 && s.runs == 1)
                                 : s.waves == 1 && s.tiles == 16 && (ns > 1 || s.runs == 2);
  const bool runs = s.runs == 1 || (s.runs == 2 && contiguous);
  if (!held || !runs || s.blocks_per_cu < 0 || threads == 0 || threads > UINT32_MAX) {
    fprintf(stderr, "%d entries, %d segments, %u vectors of %d: %d waves, %llu threads\n", ns,
            ncover, n_vec, vec, s.waves, (unsigned long long)threads);
    exit(1);
  }
}

static void check_lds() {
  constexpr int kCu = 160 << 10, kUnit = kLdsUnit;
  // The tuning interface's cap: as many blocks as hold that many waves.
  for (int per_block : {1, 4})
    for (int waves = -1; waves <= 32; ++waves) {
      const int blocks = waves < per_block ? 1 : waves / per_block;
      const size_t lds = occupancy_lds(kCu, waves, per_block);
      const size_t taken = (lds + kUnit - 1) / kUnit * kUnit;
      const bool capped = waves > 0 && blocks >= 3 && blocks * per_block < 32;
      if ((lds != 0) != capped ||
          (capped && (taken * blocks > size_t(kCu) ||
                      (blocks <= 12 && taken * (blocks + 1) <= size_t(kCu))))) {
        fprintf(stderr, "%d waves in blocks of %d: %zu reserved\n", waves, per_block, lds);
        exit(1);
      }
    }
  for (int blocks = 0; blocks <= 32; ++blocks)
    for (size_t own = 0; own <= 64u << 10; own += 512) {
      const size_t extra = residual_lds(kCu, blocks, own, 0), all = own + extra;
      const size_t taken = (all + kUnit - 1) / kUnit * kUnit;
      const bool fits = extra == 0 || (all <= 64u << 10 && taken * blocks <= size_t(kCu) &&
                                       (blocks > 12 || taken * (blocks + 1) > size_t(kCu)));
      if (!fits || residual_lds(kCu, blocks, own, -1) != 0 ||
          residual_lds(kCu, blocks, own, 7) != extra) {
        fprintf(stderr, "%d blocks, own LDS %zu: %zu reserved\n", blocks, own, extra);
        exit(1);
      }
    }
}

static void check_stream(int ns, int no, uint32_t n_vec) {
  for (int interleaved = 0; interleaved < 2; ++interleaved) {
    const StreamShape s = stream_shape(ns, no, interleaved != 0, n_vec, 256);
    const bool two = s.runs == 2 && !interleaved && takes_pairs(ns, no);
    if ((s.runs != 1 && !two) || s.blocks_per_cu < 0 ||
        (s.blocks_per_cu == 0 && (ns > 2 || no > 1))) {
      fprintf(stderr, "%d entries, %d outputs, %u vectors: %d runs, %d blocks\n", ns, no, n_vec,
              s.runs, s.blocks_per_cu);
      exit(1);
    }
  }
}

int main() {
  check_lds();
  for (int ns = 1; ns <= 8; ++ns)
    for (int no = 1; no <= 8; ++no)
      for (uint32_t n_vec : {0u, 1u, 1u << 15, 1u << 20, 1u << 25, (1u << 31) - 1})
        check_stream(ns, no, n_vec);
  const uint32_t sizes[] = {1, 64, 65, 1u << 14, 5u << 14, 9u << 14, 13u << 14, 17u << 14,
                            20u << 14, 28u << 14, 40u << 14, 1u << 20, 80u << 14, 1u << 25,
                            (1u << 28) - 64, 1u << 28,
                            1u << 29, (1u << 30) - 64, (1u << 30) - 1, 1u << 30,
                            (1u << 30) + 1, (1u << 31) - 65, (1u << 31) - 1};
  for (int ns = 1; ns <= 8; ++ns)
    for (int vec = 4; vec <= 8; vec += 4)
      for (int ncover = 0; ncover <= 128; ++ncover)
        for (uint32_t n_vec : sizes)
          for (int contiguous = ns == 1; contiguous < 2; ++contiguous)
            check_grid(ns, vec, ncover, n_vec, contiguous != 0);
  printf("shapes ok\n");
  return 0;
}
