// Device kernels of libcheb for gfx950 (CDNA4, wave64).
//
// 1. The skipped-step prediction (paper, Section 3.3, forward application
//    equation; Algorithm 1, extrapolation branch): out = sum_k w_k H_k over
//    the flattened feature cache, for one target or for several targets at
//    once (all of them depend on the same history).  Pure streaming work:
//    (n+1) x 16 bytes of HBM traffic per 16-byte output vector and 2n flops
//    per element, far below the fp32 ridge point, so the kernel is laid out
//    for bandwidth: 128-bit coalesced loads (a wave covers 1 KiB contiguous
//    per load instruction), all of a thread's loads issued before any
//    arithmetic, weights as kernel arguments (they live in SGPRs), fp32
//    accumulation for bf16 and fp16 storage and fp64 for fp32 storage, and
//    one hardware round-to-nearest-even pack per element pair
//    (v_cvt_pk_bf16_f32, v_cvt_pk_f16_f32).  No LDS: nothing is reused
//    across lanes.
// 2. The full-step push (Algorithm 1, full computation: store (s, f_s) in
//    the history): a launch copies up to 64 segments into a
//    slot.
// 3. Residual application on a skipped step (Section 3.1, block equation):
//    the block stack's sum of predicted module outputs added to the
//    residual stream in one pass.
// History entries are either contiguous slots or chunk-interleaved lanes
// (internal.h): vector v of an entry is at (v / 2048) * super + v % 2048
// from the entry's base, which is v itself when super is 2048.  One-wave
// tiles make that place uniform, so it is scalar arithmetic.
#include <hip/hip_runtime.h>

#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <type_traits>

#include "internal.h"
#include "shapes.h"
#include "tiles.h"

namespace cheb {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

template <bool NT>
__device__ __forceinline__ u32x4 load16(const u32x4 *p) {
  if constexpr (NT) return __builtin_nontemporal_load(p);
  else return *p;
}

template <bool NT>
__device__ __forceinline__ void store16(u32x4 *p, u32x4 v) {
  if constexpr (NT) __builtin_nontemporal_store(v, p);
  else *p = v;
}

// History pointers (oldest to newest), output pointers and one weight row
// per output, passed by value as kernel arguments (they land in SGPRs).
// `super` is the entries' chunk stride in vectors (kChunkVecs: contiguous).
template <int NS, int NO, typename W>
struct Hist {
  const u32x4 *p[NS];
  u32x4 *o[NO];
  W w[NO][NS];
  uint64_t super;
};

// Vector v of an interleaved entry, relative to the entry's base.
__device__ __forceinline__ uint64_t lane_vec(uint64_t v, uint64_t super) {
  return (v >> kChunkShift) * super + (v & uint64_t(kChunkVecs - 1));
}

// Ragged end of a stateless combination: `count` (< elements per vector)
// trailing elements starting at element `first`, done by block 0.
struct Tail {
  uint32_t count;
  uint64_t first;
};

// ---- bfloat16 storage, fp32 accumulation ---------------------------------

struct Bf16Op {
  using W = float;
  using E = uint16_t;

  __device__ __forceinline__ static float lo(uint32_t word) {
    return __uint_as_float(word << 16);  // element 2q (low half)
  }
  __device__ __forceinline__ static float hi(uint32_t word) {
    return __uint_as_float(word & 0xffff0000u);  // element 2q+1
  }

  template <int NS>
  __device__ __forceinline__ static u32x4 vec(const u32x4 (&v)[NS], const W (&w)[NS]) {
    float a[8];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      a[2 * q] = w[0] * lo(v[0][q]);
      a[2 * q + 1] = w[0] * hi(v[0][q]);
    }
#pragma unroll
    for (int k = 1; k < NS; ++k) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        a[2 * q] = fmaf(w[k], lo(v[k][q]), a[2 * q]);
        a[2 * q + 1] = fmaf(w[k], hi(v[k][q]), a[2 * q + 1]);
      }
    }
    u32x4 r;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      f32x2 pair = {a[2 * q], a[2 * q + 1]};
      r[q] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pair, bf16x2));
    }
    return r;
  }

  template <int NS>
  __device__ __forceinline__ static E scalar(const E *const (&p)[NS], const W (&w)[NS],
                                             uint64_t i) {
    float a = w[0] * __uint_as_float(uint32_t(p[0][i]) << 16);
#pragma unroll
    for (int k = 1; k < NS; ++k) a = fmaf(w[k], __uint_as_float(uint32_t(p[k][i]) << 16), a);
    return __builtin_bit_cast(uint16_t, static_cast<__bf16>(a));
  }
};

// ---- binary16 storage, fp32 accumulation ---------------------------------

struct F16Op {
  using W = float;
  using E = uint16_t;

  __device__ __forceinline__ static f32x2 pair(uint32_t word) {  // elements 2q, 2q+1
    return __builtin_convertvector(__builtin_bit_cast(f16x2, word), f32x2);
  }

  template <int NS>
  __device__ __forceinline__ static u32x4 vec(const u32x4 (&v)[NS], const W (&w)[NS]) {
    float a[8];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x2 p = pair(v[0][q]);
      a[2 * q] = w[0] * p.x;
      a[2 * q + 1] = w[0] * p.y;
    }
#pragma unroll
    for (int k = 1; k < NS; ++k) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x2 p = pair(v[k][q]);
        a[2 * q] = fmaf(w[k], p.x, a[2 * q]);
        a[2 * q + 1] = fmaf(w[k], p.y, a[2 * q + 1]);
      }
    }
    u32x4 r;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      f32x2 pr = {a[2 * q], a[2 * q + 1]};
      r[q] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pr, f16x2));
    }
    return r;
  }

  template <int NS>
  __device__ __forceinline__ static E scalar(const E *const (&p)[NS], const W (&w)[NS],
                                             uint64_t i) {
    float a = w[0] * float(__builtin_bit_cast(_Float16, p[0][i]));
#pragma unroll
    for (int k = 1; k < NS; ++k) a = fmaf(w[k], float(__builtin_bit_cast(_Float16, p[k][i])), a);
    return __builtin_bit_cast(uint16_t, static_cast<_Float16>(a));
  }
};

// ---- binary32 storage, fp64 accumulation ---------------------------------

struct F32Op {
  using W = double;
  using E = float;

  template <int NS>
  __device__ __forceinline__ static u32x4 vec(const u32x4 (&v)[NS], const W (&w)[NS]) {
    double a[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) a[q] = w[0] * double(__uint_as_float(v[0][q]));
#pragma unroll
    for (int k = 1; k < NS; ++k)
#pragma unroll
      for (int q = 0; q < 4; ++q) a[q] = fma(w[k], double(__uint_as_float(v[k][q])), a[q]);
    u32x4 r;
#pragma unroll
    for (int q = 0; q < 4; ++q) r[q] = __float_as_uint(float(a[q]));
    return r;
  }

  template <int NS>
  __device__ __forceinline__ static E scalar(const E *const (&p)[NS], const W (&w)[NS],
                                             uint64_t i) {
    double a = w[0] * double(p[0][i]);
#pragma unroll
    for (int k = 1; k < NS; ++k) a = fma(w[k], double(p[k][i]), a);
    return float(a);
  }
};

// ---- the streaming kernels -------------------------------------------------
//
// The default: one-wave blocks, each a tile of R runs of 64 vectors, so every
// load or store instruction covers 1 KiB contiguous.  A run's place in the
// history is uniform (a chunk holds 32 runs, none crosses one), so it is
// scalar arithmetic and a load takes a scalar base and the lane's offset.  A
// scheduling barrier keeps all NS x R loads ahead of the arithmetic.  With NO
// > 1 the loaded history feeds NO weight rows and NO outputs: every skipped
// step between two full steps is predicted in one pass.  Bound by HBM: NS KiB
// read and NO KiB written per run and next to no arithmetic; how many blocks
// share a compute unit and how far a tile's runs lie apart (stream_shape)
// decide how well reads and writes mix.  The ragged tail, which only
// contiguous sources have, is a block of its own past the tiles; that block's
// runs never count as whole (whole_tile), so whole tiles go without a test
// for it (one ahead of it, or in 64 bits, costs 2 to 5% with 3 contiguous
// entries: of 1 GB in bf16, 573 us -> 599).
template <class Op, int NS, int NO, int R, bool NT>
__global__ __launch_bounds__(64) void stream_kernel(Hist<NS, NO, typename Op::W> h, uint32_t n_vec,
                                                    uint32_t n_tiles, uint32_t lg, Tail tail) {
  const uint32_t lane = threadIdx.x;
  const RunTile tile = run_tile<R>(blockIdx.x, n_vec, lg);
  if (whole_tile<R>(tile, n_vec)) {
    u32x4 v[R][NS];
#pragma unroll
    for (int k = 0; k < NS; ++k)
#pragma unroll
      for (int r = 0; r < R; ++r)
        v[r][k] = load16<NT>(h.p[k] + lane_vec(tile.first + uint32_t(r) * tile.stride, h.super) +
                             lane);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int m = 0; m < NO; ++m)
#pragma unroll
      for (int r = 0; r < R; ++r)
        store16<NT>(h.o[m] + tile.first + uint32_t(r) * tile.stride + lane,
                    Op::template vec<NS>(v[r], h.w[m]));
    return;
  }
  if (blockIdx.x == n_tiles) {
    if (lane >= tail.count) return;
    using E = typename Op::E;
    const E *p[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k) p[k] = reinterpret_cast<const E *>(h.p[k]);
    const uint64_t i = tail.first + lane;
#pragma unroll
    for (int m = 0; m < NO; ++m)
      reinterpret_cast<E *>(h.o[m])[i] = Op::template scalar<NS>(p, h.w[m], i);
    return;
  }
#pragma unroll 1
  for (int r = 0; r < R; ++r) {
    const uint32_t first = tile.first + uint32_t(r) * tile.stride;
    if (first + lane >= n_vec) return;
    u32x4 v[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k) v[k] = load16<NT>(h.p[k] + lane_vec(first, h.super) + lane);
#pragma unroll
    for (int m = 0; m < NO; ++m)
      store16<NT>(h.o[m] + first + lane, Op::template vec<NS>(v, h.w[m]));
  }
}

// The other launch shapes of the tuning interface.  The vector range
// [0, n_vec) is cut into tiles of BLK * U vectors.  A block takes tiles
// blockIdx.x, blockIdx.x + gridDim.x, ... (one tile per block when the grid
// covers the range, a persistent loop otherwise).  In a tile, lane t handles
// vectors t, t + BLK, ..., so every load instruction of a wave reads 64
// consecutive 16-byte vectors (1 KiB), all NS x U of them ahead of its
// arithmetic.
template <class Op, int NS, int NO, int BLK, int U, bool NT>
__global__ __launch_bounds__(BLK) void combine_kernel(Hist<NS, NO, typename Op::W> h,
                                                      uint32_t n_vec, uint32_t n_tiles,
                                                      Tail tail) {
  const bool flat = h.super == uint64_t(kChunkVecs);
  for (uint32_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
    const uint32_t base = tile * uint32_t(BLK * U) + threadIdx.x;
    if (base + uint32_t((U - 1) * BLK) < n_vec) {
      u32x4 v[U][NS];
      if (flat) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int k = 0; k < NS; ++k) v[u][k] = load16<NT>(h.p[k] + base + u * BLK);
      } else {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const uint64_t off = lane_vec(base + u * BLK, h.super);
#pragma unroll
          for (int k = 0; k < NS; ++k) v[u][k] = load16<NT>(h.p[k] + off);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int m = 0; m < NO; ++m)
          store16<NT>(h.o[m] + base + u * BLK, Op::template vec<NS>(v[u], h.w[m]));
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t i = base + u * BLK;
        if (i < n_vec) {
          const uint64_t off = flat ? uint64_t(i) : lane_vec(i, h.super);
          u32x4 v[NS];
#pragma unroll
          for (int k = 0; k < NS; ++k) v[k] = load16<NT>(h.p[k] + off);
#pragma unroll
          for (int m = 0; m < NO; ++m) store16<NT>(h.o[m] + i, Op::template vec<NS>(v, h.w[m]));
        }
      }
    }
  }
  // A ragged tail only exists for contiguous sources (the host ensures it).
  if (tail.count != 0 && blockIdx.x == 0 && threadIdx.x < tail.count) {
    using E = typename Op::E;
    const E *p[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k) p[k] = reinterpret_cast<const E *>(h.p[k]);
    const uint64_t i = tail.first + threadIdx.x;
#pragma unroll
    for (int m = 0; m < NO; ++m)
      reinterpret_cast<E *>(h.o[m])[i] = Op::template scalar<NS>(p, h.w[m], i);
  }
}

// The device the launch goes to.
struct Gpu {
  int cus;         // compute units
  int lds_per_cu;  // LDS bytes per compute unit
  int waves;       // occupancy cap in waves per compute unit, 0: none (of the
                   // residual kernel: as configured, and only -1 counts)
};

// Waves per compute unit of the other launch shapes, whose loops and larger
// blocks came out best at 44 KiB of loads in flight (one output) and 36
// (several).
int auto_waves(int ns, int no) {
  if (ns <= 2) return 0;
  const int kib = no == 1 ? 44 : 36;
  return std::max(6, (kib + ns / 2) / ns);
}

template <class Op, int NS, int NO, int BLK, int U, bool NT>
hipError_t launch_shape(const Hist<NS, NO, typename Op::W> &h, uint32_t n_vec, Tail tail,
                        int blocks_per_cu, const Gpu &g, hipStream_t s) {
  const uint32_t per_tile = uint32_t(BLK * U);
  const uint32_t n_tiles = (n_vec + per_tile - 1) / per_tile;
  uint32_t grid = std::max<uint32_t>(n_tiles, 1u);
  if (blocks_per_cu > 0) grid = std::min<uint32_t>(grid, uint32_t(blocks_per_cu) * uint32_t(g.cus));
  hipLaunchKernelGGL((combine_kernel<Op, NS, NO, BLK, U, NT>), dim3(grid), dim3(BLK),
                     occupancy_lds(g.lds_per_cu, g.waves, BLK / 64), s, h, n_vec, n_tiles, tail);
  return hipGetLastError();
}

// The default launch shape.
template <class Op, int NS, int NO, int R, bool NT>
hipError_t launch_runs(const Hist<NS, NO, typename Op::W> &h, uint32_t n_vec, Tail tail,
                       int blocks, uint32_t lg, const Gpu &g, hipStream_t s) {
  const uint32_t tiles = run_tiles<R>(n_vec, lg);
  hipLaunchKernelGGL((stream_kernel<Op, NS, NO, R, NT>), dim3(tiles + (tail.count != 0 ? 1u : 0u)),
                     dim3(64), blocks > 2 && blocks < 32 ? lds_share(g.lds_per_cu, blocks) : 0, s,
                     h, n_vec, tiles, lg, tail);
  return hipGetLastError();
}

template <class Op, int NS, int NO, bool NT>
hipError_t launch_stream(const Hist<NS, NO, typename Op::W> &h, uint32_t n_vec, Tail tail,
                         const cheb_launch_config &cfg, const Gpu &g, hipStream_t s) {
  if constexpr (NT) {
    if (cfg.waves_per_cu == 0) {
      const StreamShape shape =
          stream_shape(NS, NO, h.super != uint64_t(kChunkVecs), n_vec, g.cus);
      if constexpr (takes_pairs(NS, NO))
        if (shape.runs == 2)
          return launch_runs<Op, NS, NO, 2, NT>(h, n_vec, tail, shape.blocks_per_cu, kPairLg, g,
                                                s);
      return launch_runs<Op, NS, NO, 1, NT>(h, n_vec, tail, shape.blocks_per_cu, kRunLg, g, s);
    }
  }
  return launch_runs<Op, NS, NO, 1, NT>(h, n_vec, tail, g.waves, kRunLg, g, s);
}

// Single output: every launch shape of the tuning interface.
template <class Op, int NS, bool NT>
hipError_t launch_one(const Hist<NS, 1, typename Op::W> &h, uint32_t n_vec, Tail tail,
                      const cheb_launch_config &cfg, const Gpu &dev, hipStream_t s) {
  const int b = cfg.block, u = cfg.unroll, g = cfg.blocks_per_cu;
  // A problem too small to give every compute unit a few 1024-thread blocks
  // runs with 256-thread blocks instead (four times as many blocks).
  const bool small = uint64_t(n_vec) < uint64_t(4 * 1024) * uint64_t(dev.cus);
  if (b == 64 && g == 0) return launch_stream<Op, NS, 1, NT>(h, n_vec, tail, cfg, dev, s);
  if (b == 64) return launch_shape<Op, NS, 1, 64, 1, NT>(h, n_vec, tail, g, dev, s);
  if (b == 1024 && small) return launch_shape<Op, NS, 1, 256, 1, NT>(h, n_vec, tail, g, dev, s);
  if (b == 1024) return launch_shape<Op, NS, 1, 1024, 1, NT>(h, n_vec, tail, g, dev, s);
  if (b == 512) {
    if (u == 1) return launch_shape<Op, NS, 1, 512, 1, NT>(h, n_vec, tail, g, dev, s);
    return launch_shape<Op, NS, 1, 512, 2, NT>(h, n_vec, tail, g, dev, s);
  }
  if (u == 1) return launch_shape<Op, NS, 1, 256, 1, NT>(h, n_vec, tail, g, dev, s);
  if (u == 2) return launch_shape<Op, NS, 1, 256, 2, NT>(h, n_vec, tail, g, dev, s);
  return launch_shape<Op, NS, 1, 256, 4, NT>(h, n_vec, tail, g, dev, s);
}

// Several outputs: one vector per lane, a grid covering the range, 64-lane
// blocks or 1024-lane blocks for any other configured block, and the
// non-temporal hint as configured; this keeps the number of kernel instances
// bounded.
template <class Op, int NS, int NO>
hipError_t launch_many(const Hist<NS, NO, typename Op::W> &h, uint32_t n_vec, Tail tail,
                       const cheb_launch_config &cfg, const Gpu &dev, hipStream_t s) {
  if (cfg.block == 64)
    return cfg.nontemporal ? launch_stream<Op, NS, NO, true>(h, n_vec, tail, cfg, dev, s)
                           : launch_stream<Op, NS, NO, false>(h, n_vec, tail, cfg, dev, s);
  return cfg.nontemporal ? launch_shape<Op, NS, NO, 1024, 1, true>(h, n_vec, tail, 0, dev, s)
                         : launch_shape<Op, NS, NO, 1024, 1, false>(h, n_vec, tail, 0, dev, s);
}

template <class Op, int NS, int NO>
hipError_t launch_ns_no(const void *const *src, const double *w, void *const *out,
                        int64_t numel, int64_t super_vecs, const cheb_launch_config &cfg,
                        const Gpu &dev0, hipStream_t s) {
  constexpr int kVec = 16 / int(sizeof(typename Op::E));
  Gpu dev = dev0;
  Hist<NS, NO, typename Op::W> h;
  h.super = uint64_t(super_vecs);
  for (int k = 0; k < NS; ++k) h.p[k] = static_cast<const u32x4 *>(src[k]);
  for (int m = 0; m < NO; ++m) {
    h.o[m] = static_cast<u32x4 *>(out[m]);
    for (int k = 0; k < NS; ++k) h.w[m][k] = static_cast<typename Op::W>(w[m * NS + k]);
  }
  const uint32_t n_vec = uint32_t(numel / kVec);
  if (cfg.waves_per_cu != 0)
    dev.waves = std::max(0, cfg.waves_per_cu);
  else if (cfg.block == 64 && cfg.blocks_per_cu == 0)
    dev.waves = single_blocks(NS, NO, super_vecs != kChunkVecs, n_vec, dev.cus);
  else
    dev.waves = auto_waves(NS, NO);
  Tail tail{uint32_t(numel % kVec), uint64_t(numel / kVec) * kVec};
  if constexpr (NO == 1) {
    return cfg.nontemporal ? launch_one<Op, NS, true>(h, n_vec, tail, cfg, dev, s)
                           : launch_one<Op, NS, false>(h, n_vec, tail, cfg, dev, s);
  } else {
    return launch_many<Op, NS, NO>(h, n_vec, tail, cfg, dev, s);
  }
}

template <class Op, int NS>
hipError_t launch_ns(const void *const *src, const double *w, int n_out, void *const *out,
                     int64_t numel, int64_t sv, const cheb_launch_config &cfg, const Gpu &cus,
                     hipStream_t s) {
  switch (n_out) {
    case 1: return launch_ns_no<Op, NS, 1>(src, w, out, numel, sv, cfg, cus, s);
    case 2: return launch_ns_no<Op, NS, 2>(src, w, out, numel, sv, cfg, cus, s);
    case 3: return launch_ns_no<Op, NS, 3>(src, w, out, numel, sv, cfg, cus, s);
    case 4: return launch_ns_no<Op, NS, 4>(src, w, out, numel, sv, cfg, cus, s);
    case 5: return launch_ns_no<Op, NS, 5>(src, w, out, numel, sv, cfg, cus, s);
    case 6: return launch_ns_no<Op, NS, 6>(src, w, out, numel, sv, cfg, cus, s);
    case 7: return launch_ns_no<Op, NS, 7>(src, w, out, numel, sv, cfg, cus, s);
    default: return launch_ns_no<Op, NS, 8>(src, w, out, numel, sv, cfg, cus, s);
  }
}

template <class Op>
hipError_t launch_op(const void *const *src, int n, const double *w, int n_out,
                     void *const *out, int64_t numel, int64_t sv,
                     const cheb_launch_config &cfg, const Gpu &cus, hipStream_t s) {
  switch (n) {
    case 1: return launch_ns<Op, 1>(src, w, n_out, out, numel, sv, cfg, cus, s);
    case 2: return launch_ns<Op, 2>(src, w, n_out, out, numel, sv, cfg, cus, s);
    case 3: return launch_ns<Op, 3>(src, w, n_out, out, numel, sv, cfg, cus, s);
    case 4: return launch_ns<Op, 4>(src, w, n_out, out, numel, sv, cfg, cus, s);
    case 5: return launch_ns<Op, 5>(src, w, n_out, out, numel, sv, cfg, cus, s);
    case 6: return launch_ns<Op, 6>(src, w, n_out, out, numel, sv, cfg, cus, s);
    case 7: return launch_ns<Op, 7>(src, w, n_out, out, numel, sv, cfg, cus, s);
    default: return launch_ns<Op, 8>(src, w, n_out, out, numel, sv, cfg, cus, s);
  }
}

// ---- full-step push: segment gather into one slot --------------------------

constexpr uint32_t kGatherTile = uint32_t(kGatherTileVecs);  // vectors per block, one per lane

struct GatherArgs {
  const void *src[kGatherSegs];
  uint64_t dst_vec[kGatherSegs];  // vectors from the entry's base
  uint64_t numel[kGatherSegs];
  GatherClass cls[kGatherClasses];
  int32_t classes;
};

// Flat: x = tile of a segment, y = segment; blocks past their segment's end
// return at once.  In classes a block finds its own by a scan of at most 16 and
// its segment there by a division, both scalar (next_gather).  Bound by HBM, half
// reads and half writes: one-wave blocks at full occupancy mix the two best
// (FLUX-1024 into a contiguous slot: 485 us, 6.6 TB/s, against 514 with 256-lane
// blocks and 500 or more with two or four vectors per lane at any limit on
// resident blocks; into an interleaved lane 525 against 548).  Source reads and
// slot writes are streaming (each byte is touched once per push), so both carry
// the non-temporal hint.  For interleaved entries tiles are whole in the entry,
// not in the segment (a segment's first one may begin with idle lanes), so a tile
// lies in one chunk and its place is uniform, and one that straddled 128-byte
// lines would share them with its neighbours, which run on other XCDs (6 fp32
// segments of 41 MB that start anywhere in a line, into one of six lanes: 82 us
// against 89 with tiles cut from the segment's start).  In contiguous slots whose
// segments all start on 64 bytes they are cut from the segment's start, which
// spares a load at the head of each block and lets the reads start on a line (DiT
// steps of 10 to 30 us 1.5 to 2.3% faster, 36 fp32 tensors of 57 MB 639 us -> 622).
template <typename E, bool kFlat, bool kWhole>  // kWhole: tiles whole in the entry
__global__ __launch_bounds__(64) void gather_kernel(GatherArgs a, char *__restrict__ slot,
                                                    uint64_t super) {
  constexpr int kVec = 16 / int(sizeof(E));
  uint32_t s = blockIdx.y, tile = blockIdx.x;
  if constexpr (!kFlat) {
    int32_t p = 0;
    for (int32_t q = 1; q < a.classes; ++q)
      if (blockIdx.x >= a.cls[q].block) p = q;
    const GatherClass c = a.cls[p];
    const uint32_t b = blockIdx.x - c.block;
    s = __umulhi(b, c.inverse);  // b / tiles, or one less
    tile = b - s * c.tiles;
    if (tile >= c.tiles) {
      ++s;
      tile -= c.tiles;
    }
    s += uint32_t(c.seg);
  }
  const uint64_t numel = a.numel[s];
  const uint32_t n_full = uint32_t(numel / kVec);
  const uint32_t rem = uint32_t(numel % kVec);
  const uint32_t lead = kWhole ? uint32_t(a.dst_vec[s]) & (kGatherTile - 1) : 0u;
  const uint32_t first = tile * kGatherTile;
  const uint32_t lane = threadIdx.x;
  if (first > n_full + lead) return;
  u32x4 *dst = reinterpret_cast<u32x4 *>(slot) +
               lane_vec(a.dst_vec[s] - lead + first, super) + lane;
  const uint32_t i = first + lane - lead;  // wraps to past any segment before its first vector
  const u32x4 *src = static_cast<const u32x4 *>(a.src[s]) + i;
  if (i < n_full) {
    store16<true>(dst, load16<true>(src));
  } else if (i == n_full && rem != 0) {
    // Last, partial vector: copy the remaining elements one by one and zero
    // the padding up to the 16-byte boundary.
    const E *src_e = reinterpret_cast<const E *>(src);
    E tmp[kVec];
#pragma unroll
    for (int e = 0; e < kVec; ++e) tmp[e] = uint32_t(e) < rem ? src_e[e] : E(0);
    u32x4 packed;
    memcpy(&packed, tmp, 16);
    *dst = packed;
  }
}

// ---- residual application on a skipped step ---------------------------------
//
// A DiT block adds its module outputs to the residual stream (Section 3.1,
// block equation).  When every module output of a step is predicted, the
// block stack adds sum_k w_k H_k[segment] for every cached segment, so
//     x_out[j] = x_in[j] + sum_{segments s covering j} sum_k w_k H_k[s, j]
// can be formed in one pass that reads the history once and never writes
// the per-module predictions.  A launch covers the intervals of the residual
// on which the set of covering segments is constant (all of it for DiT; the
// text and image parts for FLUX), as many as its tables hold.  The covering
// segments travel as vector offsets in the kernel arguments: residual vector
// j takes vector delta[s] + j of the entry at base[k].  Accumulation is fp64
// (hundreds of terms per element), output fp32.

struct Bf16Dec {
  static constexpr int kVec = 8;
  __device__ __forceinline__ static void add(double (&a)[8], u32x4 v, double w) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      a[2 * q] = fma(w, double(__uint_as_float(v[q] << 16)), a[2 * q]);
      a[2 * q + 1] = fma(w, double(__uint_as_float(v[q] & 0xffff0000u)), a[2 * q + 1]);
    }
  }
};

struct F16Dec {
  static constexpr int kVec = 8;
  __device__ __forceinline__ static void add(double (&a)[8], u32x4 v, double w) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const f32x2 p = F16Op::pair(v[q]);
      a[2 * q] = fma(w, double(p.x), a[2 * q]);
      a[2 * q + 1] = fma(w, double(p.y), a[2 * q + 1]);
    }
  }
};

struct F32Dec {
  static constexpr int kVec = 4;
  __device__ __forceinline__ static void add(double (&a)[4], u32x4 v, double w) {
#pragma unroll
    for (int q = 0; q < 4; ++q) a[q] = fma(w, double(__uint_as_float(v[q])), a[q]);
  }
};

constexpr int kResCover = 128;
constexpr int kResIntervals = kMaxResIntervals;

// One interval's part of a launch: tiles from `tile` on.
struct ResPart {
  uint32_t tile;
  uint32_t vec_begin, n_vec;
  int32_t first, ncover;  // its covering segments in the delta table
};

template <int NS>
struct ResArgs {
  uint64_t base[NS];
  double w[NS];
  int64_t delta[kResCover];  // vectors, from an entry's base to the segment's residual vector 0
  ResPart part[kResIntervals];
  int32_t n_part;
  uint32_t n_tiles;
  const float *x_in;  // may be null: zero
  float *x_out;
  uint64_t super;
};

// A tile's vectors of one covering segment: entry k's of run i go to v[i][k].
// The place of a run's first vector is uniform (scalar arithmetic); a lane
// adds its own index and, past the end of that vector's chunk, the jump to
// the entry's next one (64 vectors span at most two chunks; for contiguous
// entries super is kChunkVecs and there is no jump).
template <int NS, int T>
__device__ __forceinline__ void res_load(u32x4 (&v)[T][NS], const ResArgs<NS> &a, uint64_t delta,
                                         const uint64_t (&j0)[T], const uint32_t (&lane)[T]) {
  uint64_t at[T];
  uint32_t l[T];
#pragma unroll
  for (int i = 0; i < T; ++i) {
    const uint64_t v0 = delta + j0[i];
    const uint32_t r = uint32_t(v0) & uint32_t(kChunkVecs - 1);
    at[i] = ((v0 >> kChunkShift) * a.super + r) * 16u;
    l[i] = lane[i] +
           (r + lane[i] >= uint32_t(kChunkVecs) ? uint32_t(a.super - uint64_t(kChunkVecs)) : 0u);
  }
#pragma unroll
  for (int k = 0; k < NS; ++k)
#pragma unroll
    for (int i = 0; i < T; ++i) {
      // In the global address space: an address made from an integer is
      // otherwise loaded as a flat one.
      auto *p = reinterpret_cast<const __attribute__((address_space(1))) char *>(a.base[k] + at[i]);
      v[i][k] = __builtin_nontemporal_load(
          reinterpret_cast<const __attribute__((address_space(1))) u32x4 *>(p + l[i] * 16u));
    }
}

// Bound by HBM reads: NS x ncover loads of 1 KiB per run of 64 residual
// vectors.  Either the W waves of a block share a tile (G = 1): they take the
// covering segments in turn, U at a time with all their loads ahead of the
// arithmetic, into fp64 partial sums of the same vectors, and add those up
// through LDS.  Dividing the segments among waves gives a small residual W
// times the waves to fill the chip with, and has the blocks in flight read
// neighbouring kilobytes of a few places at a time rather than 16 KiB runs of
// every place.  Or each of a block's G waves has a tile of its own (W = 1),
// which keeps neighbouring tiles together on a compute unit.  residual_shape
// says which.  Measured on MI355X against one residual vector per lane of
// 1024-lane blocks: the FLUX-1024 cache, 6 interleaved entries, 1566 -> 1447
// us (6.3 -> 6.8 TB/s); DiT-XL/2 256 for one image (56 segments, 1152 tiles),
// 3 entries, 66 -> 33 us; an eighth of it (144 tiles), 54 -> 10 us.
// From contiguous memory a wave reads two runs 64 KiB apart (T = 2) at once:
// kilobytes at that distance share open DRAM rows, which the many far places
// a tile reads would otherwise close between them (FLUX-1024, 6 contiguous
// entries, 1600 -> 1454 us; one entry, 292 -> 266; at 16 KiB apart 1.5 to 3%
// less, at 128 KiB nothing).  Interleaved entries have that neighbourhood
// already and lose 2% by it.
template <class Dec, int NS, int W, int G, int U, int T>
__global__ __launch_bounds__(64 * W * G) void residual_kernel(ResArgs<NS> a) {
  static_assert(W == 1 || G == 1, "waves share a tile or have one each");
  constexpr int V = Dec::kVec;
  constexpr uint32_t kThreads = 64u * W;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t own = G == 1 ? blockIdx.x : blockIdx.x * uint32_t(G) + wave;
  if (G > 1 && own >= a.n_tiles) return;
  int32_t p = 0;
  for (int32_t q = 1; q < a.n_part; ++q)
    if (own >= a.part[q].tile) p = q;
  const ResPart part = a.part[p];
  const RunTile tile = run_tile<T>(own - part.tile, part.n_vec, kPairLg);
  uint32_t live[T], l[T];  // vectors of a run; a lane's own (idle lanes repeat the last)
  uint64_t j0[T];
#pragma unroll
  for (int i = 0; i < T; ++i) {
    const uint32_t first = tile.first + uint32_t(i) * tile.stride;
    const uint32_t left = first < part.n_vec ? part.n_vec - first : 0u;
    live[i] = left < kRun ? left : kRun;
    // a run past the end reads the first one's place again
    j0[i] = uint64_t(part.vec_begin) + (left ? first : tile.first);
    const uint32_t run = left ? live[i] : live[0];
    l[i] = lane < run ? lane : run - 1u;
  }
  const int64_t *delta = a.delta + part.first;
  const int32_t nc = part.ncover;
  double acc[T][V];
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int e = 0; e < V; ++e) acc[i][e] = -0.0;  // the sum of nothing: x + -0.0 is x, -0.0 too
  u32x4 x1[W == 1 ? T * V / 4 : 1];  // one wave: the residual's own values, ahead of the history
  if constexpr (W == 1) {
#pragma unroll
    for (int h = 0; h < T * V / 4; ++h) {
      const int i = h / (V / 4);
      x1[h] = u32x4{0u, 0u, 0u, 0u};
      if (a.x_in)
        x1[h] = *(reinterpret_cast<const u32x4 *>(a.x_in + (j0[i] + l[i]) * V) + h % (V / 4));
    }
  }
  auto take = [&](auto count, int32_t at) {
    constexpr int N = decltype(count)::value;
    u32x4 v[N][T][NS];
#pragma unroll
    for (int u = 0; u < N; ++u) res_load(v[u], a, uint64_t(delta[at + u]), j0, l);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < N; ++u)
#pragma unroll
      for (int i = 0; i < T; ++i)
#pragma unroll
        for (int k = 0; k < NS; ++k) Dec::add(acc[i], v[u][i][k], a.w[k]);
  };
  int32_t c = G == 1 ? int32_t(wave) * U : 0;
  for (; c + U <= nc; c += W * U) take(std::integral_constant<int, U>(), c);
  // the last group, if it is this wave's and partial
  if constexpr (U > 2) {
    if (c + 2 <= nc) {
      take(std::integral_constant<int, 2>(), c);
      c += 2;
    }
  }
  if constexpr (U > 1) {
    for (; c < nc; ++c) take(std::integral_constant<int, 1>(), c);
  }
  if constexpr (W == 1) {
#pragma unroll
    for (int h = 0; h < T * V / 4; ++h) {
      const int i = h / (V / 4), e = h % (V / 4) * 4;
      if (lane >= live[i]) continue;
      u32x4 r;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        r[q] = __float_as_uint(float(double(__uint_as_float(x1[h][q])) + acc[i][e + q]));
      *reinterpret_cast<u32x4 *>(a.x_out + (j0[i] + lane) * V + e) = r;
    }
  } else {
    // Element e of vector n of run i at [(i * V + e) * 64 + n]: consecutive
    // lanes write consecutive words.
    __shared__ double sums[W][T * V * kRun];
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
      for (int e = 0; e < V; ++e) sums[wave][(i * V + e) * int(kRun) + lane] = acc[i][e];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < T; ++i)
      for (uint32_t h = threadIdx.x; h < live[i] * uint32_t(V / 4); h += kThreads) {
        const uint64_t o = j0[i] * V + 4u * h;
        const uint32_t at = (uint32_t(i * V) + 4u * h % V) * kRun + 4u * h / V;
        u32x4 x = {0u, 0u, 0u, 0u}, r;
        if (a.x_in) x = *reinterpret_cast<const u32x4 *>(a.x_in + o);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          double s = double(__uint_as_float(x[q]));
#pragma unroll
          for (int w = 0; w < W; ++w) s += sums[w][at + uint32_t(q) * kRun];
          r[q] = __float_as_uint(float(s));
        }
        *reinterpret_cast<u32x4 *>(a.x_out + o) = r;
      }
  }
}

// The launch's intervals with their tiles numbered through.
struct ResJob {
  const uint64_t *base;
  const double *w;
  const int64_t *delta;
  int n_delta;
  const ResidualInterval *iv;
  int n_iv;
  const float *x_in;
  float *x_out;
  uint64_t super;
};

template <class Dec, int NS>
hipError_t launch_residual_ns(const ResJob &j, const Gpu &g, hipStream_t s) {
  ResArgs<NS> a;
  memset(&a, 0, sizeof a);
  a.super = j.super;
  memcpy(a.base, j.base, sizeof a.base);
  memcpy(a.w, j.w, sizeof a.w);
  memcpy(a.delta, j.delta, sizeof(int64_t) * size_t(j.n_delta));
  a.x_in = j.x_in;
  a.x_out = j.x_out;
  a.n_part = j.n_iv;
  uint32_t singles = 0;
  int ncover = 0;
  for (int i = 0; i < j.n_iv; ++i) {
    singles += run_tiles<1>(uint32_t(j.iv[i].n_vec), kPairLg);
    ncover = std::max(ncover, int(j.iv[i].ncover));
  }
  const ResShape shape = within_grid(
      residual_shape(NS, Dec::kVec, ncover, singles, j.super == uint64_t(kChunkVecs), g.cus),
      singles);
  uint32_t tiles = 0;
  for (int i = 0, first = 0; i < j.n_iv; first += j.iv[i].ncover, ++i) {
    const uint32_t n_vec = uint32_t(j.iv[i].n_vec);
    a.part[i] = ResPart{tiles, uint32_t(j.iv[i].vec_begin), n_vec, first, j.iv[i].ncover};
    tiles += shape.runs == 2 ? run_tiles<2>(n_vec, kPairLg) : run_tiles<1>(n_vec, kPairLg);
  }
  a.n_tiles = tiles;
  auto launch = [&](auto waves, auto grouped, auto runs) {
    constexpr int W = decltype(waves)::value, G = decltype(grouped)::value;
    constexpr int T = decltype(runs)::value;
    // Segments a wave loads before its arithmetic.
    constexpr int U = G > 1       ? 2 / T
                      : NS == 1   ? 4 / T
                      : NS == 2   ? (T == 2 && W == 1 ? 1 : 2)
                                  : 1;
    constexpr size_t kOwn = W > 1 ? size_t(W) * T * kRun * Dec::kVec * sizeof(double) : 0;
    const size_t extra = residual_lds(g.lds_per_cu, shape.blocks_per_cu, kOwn, g.waves);
    hipLaunchKernelGGL((residual_kernel<Dec, NS, W, G, U, T>), dim3((tiles + G - 1) / G),
                       dim3(64 * W * G), extra, s, a);
  };
  const std::integral_constant<int, 1> one;
  const std::integral_constant<int, 2> two;
  const std::integral_constant<int, 4> four;
  const std::integral_constant<int, 16> sixteen;
  if (shape.tiles == 16) {
    if constexpr (NS == 1)  // contiguous, and never in blocks of single runs
      launch(one, sixteen, two);
    else
      shape.runs == 2 ? launch(one, sixteen, two) : launch(one, sixteen, one);
  } else if (shape.waves == 16)
    launch(sixteen, one, one);
  else if (shape.waves == 4)
    shape.runs == 2 ? launch(four, one, two) : launch(four, one, one);
  else if (shape.waves == 2)
    shape.runs == 2 ? launch(two, one, two) : launch(two, one, one);
  else
    shape.runs == 2 ? launch(one, one, two) : launch(one, one, one);
  return hipGetLastError();
}

template <class Dec>
hipError_t launch_residual_dec(int n, const ResJob &j, const Gpu &g, hipStream_t s) {
  switch (n) {
    case 1: return launch_residual_ns<Dec, 1>(j, g, s);
    case 2: return launch_residual_ns<Dec, 2>(j, g, s);
    case 3: return launch_residual_ns<Dec, 3>(j, g, s);
    case 4: return launch_residual_ns<Dec, 4>(j, g, s);
    case 5: return launch_residual_ns<Dec, 5>(j, g, s);
    case 6: return launch_residual_ns<Dec, 6>(j, g, s);
    case 7: return launch_residual_ns<Dec, 7>(j, g, s);
    default: return launch_residual_ns<Dec, 8>(j, g, s);
  }
}

}  // namespace

int launch_combine(int dtype, const void *const *src, int n, const double *w, int n_out,
                   void *const *out, int64_t numel, int64_t super_vecs, hipStream_t stream) {
  if (numel == 0) return ok();
  Gpu cus{0, 0, 0};
  int rc = device_info(&cus.cus, &cus.lds_per_cu);
  if (rc != CHEB_OK) return rc;
  const cheb_launch_config cfg = launch_shape();
  hipError_t e;
  switch (dtype) {
    case CHEB_BF16:
      e = launch_op<Bf16Op>(src, n, w, n_out, out, numel, super_vecs, cfg, cus, stream);
      break;
    case CHEB_F16:
      e = launch_op<F16Op>(src, n, w, n_out, out, numel, super_vecs, cfg, cus, stream);
      break;
    default:
      e = launch_op<F32Op>(src, n, w, n_out, out, numel, super_vecs, cfg, cus, stream);
      break;
  }
  if (e != hipSuccess) return fail(CHEB_E_HIP, "combine launch failed: %s", hipGetErrorString(e));
  return ok();
}

int launch_gather(int dtype, void *slot_base, GatherSeg *segs, int n_segs, int64_t super_vecs,
                  hipStream_t stream) {
  n_segs = order_segments(segs, n_segs);
  const int64_t vec = elems_per_vec(dtype);
  GatherArgs a;
  for (int at = 0; at < n_segs;) {
    const GatherPlan plan = next_gather(segs + at, n_segs - at, vec, super_vecs);
    memset(&a, 0, sizeof a);
    for (int j = 0; j < plan.segs; ++j) {
      const GatherSeg &g = segs[at + j];
      a.src[j] = g.src;
      a.dst_vec[j] = uint64_t(g.dst_offset / vec);
      a.numel[j] = uint64_t(g.numel);
    }
    memcpy(a.cls, plan.cls, sizeof(GatherClass) * size_t(plan.classes));
    a.classes = plan.classes;
    at += plan.segs;
    char *slot = static_cast<char *>(slot_base);
    const dim3 grid = plan.flat ? dim3(plan.widest, uint32_t(plan.segs)) : dim3(plan.blocks);
    auto launch = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, grid, dim3(kGatherTile), 0, stream, a, slot,
                         uint64_t(super_vecs));
      return hipGetLastError();
    };
    auto typed = [&](auto elem) {
      using E = decltype(elem);
      if (plan.whole)
        return launch(plan.flat ? gather_kernel<E, true, true> : gather_kernel<E, false, true>);
      return launch(plan.flat ? gather_kernel<E, true, false> : gather_kernel<E, false, false>);
    };
    const hipError_t e = elem_bytes(dtype) == 2 ? typed(uint16_t()) : typed(float());
    if (e != hipSuccess) return fail(CHEB_E_HIP, "push launch failed: %s", hipGetErrorString(e));
  }
  return ok();
}

int residual_max_cover() { return kResCover; }

int launch_residual_intervals(int dtype, int n, const uint64_t *base, const double *w,
                              const int64_t *delta, int n_delta, const ResidualInterval *iv,
                              int n_iv, const float *x_in, float *x_out, int64_t super_vecs,
                              hipStream_t stream) {
  Gpu g{0, 0, 0};
  int rc = device_info(&g.cus, &g.lds_per_cu);
  if (rc != CHEB_OK) return rc;
  g.waves = launch_shape().waves_per_cu;
  const ResJob j{base, w, delta, n_delta, iv, n_iv, x_in, x_out, uint64_t(super_vecs)};
  hipError_t e;
  switch (dtype) {
    case CHEB_BF16: e = launch_residual_dec<Bf16Dec>(n, j, g, stream); break;
    case CHEB_F16: e = launch_residual_dec<F16Dec>(n, j, g, stream); break;
    default: e = launch_residual_dec<F32Dec>(n, j, g, stream); break;
  }
  if (e != hipSuccess) return fail(CHEB_E_HIP, "residual launch failed: %s", hipGetErrorString(e));
  return ok();
}

int launch_residual(int dtype, int n, const uint64_t *base, const double *w, const int64_t *delta,
                    int ncover, const float *x_in, float *x_out, int64_t vec_begin,
                    int64_t n_vec, int64_t super_vecs, hipStream_t stream) {
  if (n_vec == 0) return ok();
  const ResidualInterval iv{vec_begin, n_vec, ncover};
  return launch_residual_intervals(dtype, n, base, w, delta, ncover, &iv, 1, x_in, x_out,
                                   super_vecs, stream);
}

}  // namespace cheb
