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

// LDS is handed out in units of 1280 bytes on gfx950, and a block may have 64 KiB
// of it.
constexpr int kLdsUnit = 1280, kMostLds = 64 << 10;

// Dynamic LDS a block reserves, and never touches, when `blocks` of them are
// to share a compute unit: an equal share rounded down to the unit (a size in
// between takes the next one, and one block fewer fits).  A share past what a
// block may have is cut to that, if as many blocks still fit and no more.
// Zero when there is no limit or none is possible.
inline size_t lds_share(int lds_per_cu, int blocks) {
  if (blocks <= 0 || lds_per_cu <= 0) return 0;
  const int per = lds_per_cu / blocks / kLdsUnit * kLdsUnit;
  if (per <= kMostLds) return size_t(per);
  return lds_per_cu / kMostLds == blocks ? size_t(kMostLds) : 0;
}

// The same for the prediction's other launch shapes, so that as many blocks as
// hold `waves` waves share a compute unit.  Zero when there is no cap, when the
// cap is at the hardware's own limit, or when one block would need more than
// the default 64 KiB of dynamic LDS.
inline size_t occupancy_lds(int lds_per_cu, int waves, int waves_per_block) {
  const int blocks = std::max(1, waves / waves_per_block);
  if (waves <= 0 || lds_per_cu <= 0 || blocks * waves_per_block >= 32) return 0;
  const int per = lds_per_cu / blocks / kLdsUnit * kLdsUnit;
  return per <= kMostLds ? size_t(per) : 0;
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

// The residual kernel's launch: the waves that share a tile, how many blocks
// share a compute unit, runs per tile, and tiles per block where each wave has
// one of its own.
struct ResShape {
  int waves;
  int blocks_per_cu;  // 0: no limit
  int runs = 1;
  int tiles = 1;
};

// By the sizes; cu stands for tiles of one run per compute unit.  The lines come
// from sweeps on MI355X (256 compute units) of 1 to 8 entries in bf16, both
// layouts, 1 to 57 segments and cu 0.5 to 150, of odd sizes and of models' own
// (whole multiples of 64 KiB), against the 1024-lane kernel without division
// ("lanes") as well; a line is drawn where both kinds of size gain by it.  In
// microseconds:
//  - one segment (a collapsed history) is a stream of ns reads plus the
//    residual's own read and write: one wave, about 80 KiB of those a compute
//    unit (fp32, 225K tiles: 6 entries 395 with 10 blocks, 413 without a limit;
//    8 entries 470 with 8, 495);
//  - up to 4 segments: little to divide, one wave, which needs no LDS sum (4
//    segments, 4.6K tiles, 3 entries: 14 against 16 with 4 waves), except 4 waves
//    for 5 interleaved entries or more (5 of 3 segments, cu 13.5: 13.1 against
//    13.5) and 2 or 4 where the residual is large (3 segments, 52K tiles, 2
//    entries: 89 against 91; 8 contiguous entries of 3, cu 27: 32.7 against
//    33.6; but 2 segments in fp32, whose tiles are half as large, 42 against 38);
//  - others, up to cu 4: 16 waves under one tile a compute unit (144 tiles of 56
//    segments, 3 entries: 10 against 16 with 4), else 4;
//  - to cu 8: 2 (1152 tiles of 56 segments, 3 entries: 31.9 against 33.2 with
//    4), but one for 7 or 8 contiguous entries, which have loads enough (8 of 56,
//    cu 5.2: 104 against 115), and 4 with few blocks for interleaved ones (8 of
//    56, cu 5.2: 103 against 110);
//  - about cu 10 to 16, where 16 waves a compute unit hold all tiles at once:
//    blocks of 16 tiles, one wave each, whose neighbours then stay together (8
//    contiguous entries of 8 segments, cu 13.5: 38.0, 39.2 in pairs of runs, 38.4
//    lanes; 3 interleaved of 24, cu 13.5: 42.4, 44.4 divided among 4, 42.5
//    lanes).  Past 16 a second round would run nearly empty (1.3 times the
//    time).  Not so 5 segments (8 contiguous entries, cu 13.5: 29.5, 26.7 in
//    pairs), and contiguous entries of over 12 gain nothing by it at models'
//    sizes: pairs of runs, one wave;
//  - contiguous entries to cu 24 in pairs of runs, one wave (2304 tiles of 56, 3
//    entries: 61 against 65 with 4 waves), and to 32, where 16 waves hold all
//    pairs, in blocks of 16 (3 of 24 segments, cu 27: 82.8, 86.6 in single blocks,
//    89.2 lanes; 3 of 40, cu 28.7: 151, 161.5, 160);
//  - contiguous ones beyond: up to 6 segments, and to 9 for up to 4 entries, 2
//    waves, as 5 divided among 4 leave three idle for half of the time (5 entries
//    of 5 segments, cu 43: 58.8, 69.5 with 4, 58.0 lanes); one entry of up to 31
//    single runs to cu 64 (24 segments, cu 54: 61.6 against 64.0 in pairs); the others 4
//    waves in pairs, few blocks (9072 tiles of 57 segments, 3 entries: 251 with
//    2, 262 with 4 of single runs; 15 segments, 2 entries: 84 with 4, 99 with 2;
//    FLUX-1024's reduction, one entry of 57 segments: 270 with 3, 283 with one
//    wave);
//  - interleaved ones: one or 2 waves for 2 entries of up to 12 segments (8, cu
//    27: 24.8 against 26.4 with 4), else 4, their blocks limited by the loads in
//    flight (FLUX-1024, 57 segments, 27K tiles, 6 entries: 1446 with 2 blocks,
//    1463 with 3, 1497 without a limit; 7 entries of 5, cu 42: 72.8 with 3, 80.5
//    with 2 of 8 waves).
inline ResShape residual_shape(int ns, int vec, int ncover, uint32_t tiles, bool contiguous,
                               int cus) {
  const auto upto = [&](int n) { return tiles <= uint64_t(n) * uint64_t(cus); };
  const bool few = ncover <= 4;
  if (ncover == 1 && tiles >= 32u * uint32_t(cus)) return {1, 80 / (ns + vec / 2)};
  if (ncover <= 1) return {1, 0};
  if (upto(4) && !few) return {ncover >= 16 && tiles < uint32_t(cus) ? 16 : 4, 0};
  if (upto(16) && few) {
    if (ncover == 2 || upto(4)) return {1, 0};
    if (!contiguous) return {ns >= 5 && !upto(6) ? 4 : 1, 0};
    if (upto(12) || ns == 1 || ns == 3 || ns == 4) return {1, 0};
    return ns == 2 ? ResShape{1, 0, 2} : ResShape{1, 0, 1, 16};
  }
  if (contiguous) {
    if (few) {
      if (upto(32) && ns >= 7 && ncover > 2 && !upto(24)) return {4, 0};
      if (upto(64) && (ns <= 2 || ncover == 2 || upto(32))) return {1, 0};
      if (ncover == 2 && vec == 4) return {1, 0};
      if (upto(64)) return {2, 8};
      return {2, ns >= 5 ? 4 : 0, 2};
    }
    if (upto(8)) return {ns >= 7 ? 1 : 2, 0};
    if (upto(12)) return {1, 0};
    if (upto(16)) return ncover >= 7 && ncover <= 12 && ns >= 3 ? ResShape{1, 0, 1, 16}
                                                                : ResShape{1, 0, 2};
    if (upto(24)) return {1, 0, 2};
    if (ns == 1 && ncover <= 9 && upto(64)) return {upto(32) ? 1 : 2, 0};
    if (upto(32)) return {1, 0, 2, 16};
    if (ns == 1 && ncover < 24) return {2, 0, 2};
    if (ns == 1) return ncover < 32 && upto(64) ? ResShape{4, 8} : ResShape{4, 3, 2};
    if (ncover <= 6 || (ncover <= 9 && ns <= 4)) return {2, 8};
    if (ncover <= 9) return {4, ns <= 6 || upto(64) ? 3 : 2, 2};
    if (ns >= 5) return {4, 2, 2};
    return {4, ncover < 32 ? 4 : ns == 2 ? 3 : 2, 2};
  }
  if (few) {
    if (ncover == 2 ? upto(64) : upto(ns >= 7 ? 24 : 32) || (upto(64) && ns == 2)) return {1, 0};
    if (upto(64)) return {4, ns >= 7 ? 4 : 8};
    if (ncover == 2 && vec == 4) return {1, 0};
    return {2, ns >= 7 ? 4 : ns >= 3 ? 8 : 0};
  }
  if (upto(8)) return ns >= 7 ? ResShape{4, ncover <= 6 ? 0 : 3} : ResShape{2, 0};
  if (upto(16)) {
    if (ns >= 7) return {4, ncover < 16 ? 0 : upto(10) ? 3 : 2};
    if (upto(10)) return {ns * ncover >= 120 ? 1 : 4, 0};
    return (ns <= 4 && ncover >= 7) || ncover >= 40 ? ResShape{1, 0, 1, 16} : ResShape{4, 0};
  }
  if (ncover <= 12) {
    if (ns == 2) return upto(32) ? ResShape{1, 0} : ResShape{2, 8};
    if (ns <= 4) return {4, ncover <= 6 || upto(48) ? 8 : 4};
    return {4, ns <= 6 || ncover <= 6 ? 4 : upto(64) ? 3 : 2};
  }
  if (ns <= 4 && ncover < 40 && upto(32)) return {4, ns == 2 ? 8 : 4};
  return {4, ns >= 7 || ncover >= 24 ? std::max(2, 4 - ns / 2) : 4};
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
  return {1, s.blocks_per_cu * s.waves, s.runs, s.tiles};
}

}  // namespace cheb
