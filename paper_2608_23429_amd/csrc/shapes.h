// How a launch is laid out: the prediction's and the residual kernel's blocks by
// their sizes, and the LDS that limits how many share a compute unit.  Host
// arithmetic.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "cheb.h"
#include "tiles.h"

namespace cheb {

// Dynamic LDS a block reserves, and never touches, when `blocks` of them are
// to share a compute unit: an equal share rounded down to the 1280-byte unit
// LDS is handed out in on gfx950 (a size in between takes the next unit, and
// one block fewer fits).  A share past the 64 KiB a block may have is cut to
// that, if as many blocks still fit and no more.  Zero when there is no limit
// or none is possible.
inline size_t lds_share(int lds_per_cu, int blocks) {
  constexpr int kMost = 64 << 10;
  if (blocks <= 0 || lds_per_cu <= 0) return 0;
  const int per = lds_per_cu / blocks / 1280 * 1280;
  if (per <= kMost) return size_t(per);
  return lds_per_cu / kMost == blocks ? size_t(kMost) : 0;
}

// Runs per tile and how many one-wave blocks share a compute unit (0: no
// limit) in a prediction, from the history size, the number of outputs, the
// layout and the work.  Too few blocks leave the memory latency uncovered, too
// many flood the memory queues and slow the writes.  Measured on MI355X, bf16,
// entries of 30 MB to 1.6 GB, 2 to 8 of each kind:
//  - one output: about 40 KiB of loads in flight from interleaved entries, 45
//    to 48 from contiguous ones (6 interleaved entries of 1.6 GB: 1627 us with
//    7, 1642 with 6, over 1670 with 8; 5 contiguous ones: 1417 us with 9, 1447
//    with 10);
//  - several outputs: about 60 KiB of loads and stores (2 interleaved entries,
//    5 outputs: 9 blocks, 6% less time than 12), and not below 6 to 8 (8
//    interleaved entries, 4 or 5 outputs: 7, 1% less than 6); one block less
//    for two outputs of 6 or 8 interleaved entries (8: 2.5%);
//  - a call of under 512 KiB a compute unit is over before the queues fill
//    and wants twice as many (6 entries of 9 MB: 11.4 us with 16, 12.6 with
//    7);
//  - above that, contiguous entries in tiles of two runs 64 KiB apart, which
//    share DRAM rows: one output of 3 to 5 entries (3 of 264 MB 159 us -> 154;
//    5 of 528 MB 473 -> 467) and several outputs (2 entries, 5 outputs of 264
//    MB: 289 us -> 282; 6 entries, 3 outputs of 1.06 GB in fp16: 1452 -> 1434;
//    4 to 8 entries, 3 to 5 outputs: 1 to 3% where the entries' size is a
//    multiple of some MiB, as models' are, and -1 to 1% where it is odd), with
//    6 blocks where that is 45 KiB (4 to 6 entries, 3 outputs: 1% over 5).  Two
//    outputs of 5 entries or more gain 1 to 2.5% without, one output of 6 or
//    more 2%, one or two entries 1%; interleaved entries gain nothing by it.
struct StreamShape {
  int blocks_per_cu;  // 0: no limit
  int runs = 1;
};

constexpr uint32_t kPairLg = 12;  // pairs of runs lie 4096 vectors (64 KiB) apart

constexpr bool takes_pairs(int ns, int no) {
  return no == 1 ? ns >= 3 && ns <= 5 : no == 2 ? ns <= 4 : true;
}

inline bool large_call(int ns, int no, uint32_t n_vec, int cus) {
  return uint64_t(n_vec / kRun) * uint64_t(ns + no) >= 512u * uint64_t(cus);
}

// Blocks of single runs.
inline int single_blocks(int ns, int no, bool interleaved, uint32_t n_vec, int cus) {
  static constexpr int kOne[2][CHEB_MAX_SLOTS + 1] = {{0, 0, 0, 16, 11, 9, 8, 7, 6},
                                                      {0, 0, 0, 14, 9, 8, 7, 6, 5}};
  const int sum = ns + no;
  int blocks = kOne[interleaved][ns];
  if (no > 1) {
    const int least = sum >= 12 && (ns < 8 || !interleaved) ? 6 : sum <= 9 && !interleaved ? 8 : 7;
    blocks = std::max(least, (60 + sum / 2) / sum);
    if (interleaved && no == 2 && (ns == 6 || ns == 8)) --blocks;
  }
  return large_call(ns, no, n_vec, cus) ? blocks : 2 * blocks;
}

inline StreamShape stream_shape(int ns, int no, bool interleaved, uint32_t n_vec, int cus) {
  if (!interleaved && takes_pairs(ns, no) && large_call(ns, no, n_vec, cus)) {
    const int sum = ns + no;
    if (no == 1) return {(28 + sum / 2) / sum, 2};
    if (sum == 7 || (no == 3 && sum > 7 && sum <= 9)) return {6, 2};
    return {std::max(sum >= 14 ? 4 : 5, (36 + sum / 2) / sum), 2};
  }
  return {single_blocks(ns, no, interleaved, n_vec, cus)};
}

// Waves per block, how many of its blocks share a compute unit and runs per
// tile, from the sizes (measured on MI355X, 256 compute units, bf16 unless
// said; cu = tiles of one run per compute unit):
//  - one segment (a collapsed history) is a stream of ns reads plus the
//    residual's own read and write: one wave, about 80 KiB of those a compute
//    unit (fp32, 225K tiles: 6 entries 395 us with 10 blocks, 413 without a
//    limit; 8 entries 470 with 8, 495);
//  - up to 4 segments: little to divide.  One wave, which needs no LDS sum (4
//    segments, 4.6K tiles, 3 entries: 14 us against 16 with 4 waves); two
//    where the residual is large (3 segments, 52K tiles, 2 entries: 89 us
//    against 91; but 2 segments in fp32, whose tiles are half as large, 42
//    against 38);
//  - below that: 16 waves under one tile a compute unit (144 tiles of 56
//    segments, 3 entries: 10 us against 16 with 4), 4 under 4, 2 under 8 (1152
//    tiles, 3 entries: 31.9 us against 33.2 with 4);
//  - then contiguous entries take pairs of runs: one wave without a limit
//    under cu = 32, the first third of it with single runs (2304 tiles, 3
//    entries: 61 us against 65 with 4 waves; 6072 tiles of 24 segments, 6
//    entries: 140 against 147), and 4 waves with few blocks beyond (9072
//    tiles of 57 segments, 3 entries: 251 us with 2 blocks, 262 with 4 of
//    single runs; 15 segments, 2 entries: 84 with 4, 99 with 2), but 2 waves
//    for one entry and few segments (8 segments, 18K tiles: 35 us against 43);
//  - interleaved entries 4 waves (8 for 7 entries or more), their blocks
//    limited where there are many tiles (FLUX-1024, 57 segments, 27K tiles, 6
//    entries: 1446 us with 2 blocks, 1463 with 3, 1497 without a limit; 15
//    segments, 15K tiles, 8 entries: 281 with 2, 287 with 4).
struct ResShape {
  int waves;
  int blocks_per_cu;  // 0: no limit
  int runs = 1;
};

inline ResShape residual_shape(int ns, int vec, int ncover, uint32_t tiles, bool contiguous,
                               int cus) {
  const uint32_t per_cu = tiles / uint32_t(cus);
  if (ncover == 1 && per_cu >= 32) return {1, 80 / (ns + vec / 2)};
  if (ncover <= 1 || (ncover <= 4 && per_cu < 64)) return {1, 0};
  if (ncover == 2 && vec == 4) return {1, 0};
  if (ncover <= 4 && contiguous) return {2, ns >= 5 ? 4 : 0, 2};
  if (ncover <= 4) return {2, ns >= 7 ? 4 : ns >= 3 ? 8 : 0};
  if (per_cu < 1 && ncover >= 16) return {16, 0};
  if (per_cu < 4) return {4, 0};
  if (per_cu < 8) return {2, 0};
  if (contiguous) {
    if (per_cu < 32) return {1, 0, per_cu < 12 ? 1 : 2};
    if (ns == 1) return ncover >= 24 ? ResShape{4, 3, 2} : ResShape{2, 0, 2};
    if (ns >= 5) return {4, 2, 2};
    return {4, ncover < 32 ? 4 : ns == 2 ? 3 : 2, 2};
  }
  if (per_cu < 16) return {4, 0};
  if (ns >= 7) return {8, 2};
  return {4, ncover >= 24 ? std::max(2, 4 - ns / 2) : 4};
}

// LDS reserved on top of a block's own so that `blocks` of them share a compute
// unit.  None where the caller wants the LDS left free (waves_per_cu -1 of the
// launch shape): 1 to 4% slower, but kernels on other streams find it.
inline size_t residual_lds(int lds_per_cu, int blocks, size_t own, int waves_per_cu) {
  const size_t share = waves_per_cu < 0 ? 0 : lds_share(lds_per_cu, blocks);
  return share > own ? share - own : 0;
}

// The same shape for a launch of that many tiles of one run (half as many of
// two).  HIP refuses a grid of 2^32 threads or more, which 4 waves a tile of
// 64 vectors reach at 2^30 vectors, 8 waves at 2^29; from there on, one wave a
// tile and as many waves a compute unit.
inline ResShape within_grid(ResShape s, uint32_t tiles) {
  if (uint64_t(tiles) * uint64_t(64 * s.waves) <= UINT32_MAX) return s;
  return {1, s.blocks_per_cu * s.waves, s.runs};
}

}  // namespace cheb
