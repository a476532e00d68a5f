// Stand-ins for the device launchers of libcheb, for a host-only build of
// the library's C++ sources under AddressSanitizer / UBSan / ThreadSanitizer.
// Prediction launches always report an error (the host test programs never
// reach one with valid arguments), and so do residual launches until
// stub_residual_on_host(1): then the tables are checked and fp32 entries in
// host memory are added up as they say.  The segment-copy launcher
// goes through the real one's launches, planned by the same functions: a
// budget set by stub_gather_batches_ok() says how many succeed before one
// fails, so a push that fails part-way through them can be tested on the CPU.
// The budget starts at 0 (every copy fails).  Each launch must take 1 to 64
// segments, cover them with its classes' tiles, leave few of those without work
// and give the kernel's division the right segment.
#include <atomic>

#include "internal.h"

namespace {
std::atomic<int> g_gather_batches_ok{0};
std::atomic<int> g_residual_on_host{0}, g_residual_launches{0};
}

extern "C" void stub_gather_batches_ok(int n) { g_gather_batches_ok.store(n); }
extern "C" void stub_residual_on_host(int on) { g_residual_on_host.store(on); }
extern "C" int stub_residual_launches() { return g_residual_launches.load(); }

namespace cheb {

int launch_combine(int, const void *const *, int, const double *, int, void *const *, int64_t,
                   int64_t, hipStream_t) {
  return fail(CHEB_E_HIP, "host-only build: no device launch");
}

int launch_gather(int dtype, void *, GatherSeg *segs, int n_segs, int64_t super_vecs,
                  hipStream_t) {
  const int vec = elems_per_vec(dtype);
  n_segs = order_segments(segs, n_segs);
  for (int at = 0, launch = 0; at < n_segs; ++launch) {
    const GatherPlan p = next_gather(segs + at, n_segs - at, vec, super_vecs);
    if (p.segs < 1 || p.segs > kGatherSegs || p.classes < 1 || p.classes > kGatherClasses)
      return fail(CHEB_E_INVAL, "copy launch %d of %d segments", launch, p.segs);
    uint32_t block = 0;
    int64_t flat_idle = 0;
    for (int c = 0; c < p.classes; ++c) {
      const GatherClass &k = p.cls[c];
      const int end = c + 1 < p.classes ? p.cls[c + 1].seg : p.segs;
      int64_t idle = 0;
      if (k.block != block || (c == 0 && k.seg != 0) || end <= k.seg || k.tiles < 1)
        return fail(CHEB_E_INVAL, "copy launch %d: class %d does not follow", launch, c);
      for (int j = k.seg; j < end; ++j) {
        const GatherSeg &g = segs[at + j];
        const int64_t tail =
            gather_lead(g.dst_offset / vec, p.whole) + (g.numel + vec - 1) / vec;
        if (!p.whole && (super_vecs != kChunkVecs || g.dst_offset / vec % 4 != 0))
          return fail(CHEB_E_INVAL, "copy launch %d: a tile across chunks or sectors", launch);
        const int64_t left = int64_t(k.tiles) - (tail + kGatherTileVecs - 1) / kGatherTileVecs;
        if (g.numel <= 0 || left < 0)
          return fail(CHEB_E_INVAL, "copy launch %d does not cover segment %d", launch, j);
        idle += left;
        flat_idle += left + int64_t(p.widest) - k.tiles;
        if (p.widest < k.tiles) return fail(CHEB_E_INVAL, "copy launch %d: too narrow", launch);
        // The kernel's division, for the segment's first and last tile.
        for (uint32_t b : {uint32_t(j - k.seg) * k.tiles, uint32_t(j - k.seg + 1) * k.tiles - 1}) {
          uint32_t q = uint32_t((uint64_t(b) * k.inverse) >> 32);
          if (b - q * k.tiles >= k.tiles) ++q;
          if (q != uint32_t(j - k.seg) || b - q * k.tiles >= k.tiles)
            return fail(CHEB_E_INVAL, "copy launch %d: block %u in segment %u", launch, b, q);
        }
      }
      block += uint32_t(end - k.seg) * k.tiles;
      if (idle > 24576 && idle * 8 > int64_t(end - k.seg) * k.tiles + 8 * 64)
        return fail(CHEB_E_INVAL, "copy launch %d: %lld idle tiles", launch, (long long)idle);
    }
    if (p.flat ? flat_idle > 10240 && p.classes > 1 : flat_idle <= 10240)
      return fail(CHEB_E_INVAL, "copy launch %d: %lld idle tiles", launch, (long long)flat_idle);
    if (block != p.blocks) return fail(CHEB_E_INVAL, "copy launch %d: %u blocks", launch, block);
    if (g_gather_batches_ok.fetch_sub(1) <= 0) {
      g_gather_batches_ok.store(0);
      return fail(CHEB_E_HIP, "host-only build: copy launch %d refused", launch);
    }
    at += p.segs;
  }
  return ok();
}

int residual_max_cover() { return 128; }

int launch_residual_intervals(int dtype, int n, const uint64_t *base, const double *w,
                              const int64_t *delta, int n_delta, const ResidualInterval *iv,
                              int n_iv, const float *x_in, float *x_out, int64_t super_vecs,
                              hipStream_t) {
  if (!g_residual_on_host.load()) return fail(CHEB_E_HIP, "host-only build: no device launch");
  int covers = 0;
  for (int i = 0; i < n_iv; ++i) {
    if (iv[i].vec_begin < 0 || iv[i].n_vec <= 0 || iv[i].ncover < 0)
      return fail(CHEB_E_INVAL, "residual interval %d is malformed", i);
    for (int h = 0; h < i; ++h)
      if (iv[i].vec_begin < iv[h].vec_begin + iv[h].n_vec &&
          iv[h].vec_begin < iv[i].vec_begin + iv[i].n_vec)
        return fail(CHEB_E_INVAL, "residual intervals %d and %d overlap", h, i);
    covers += iv[i].ncover;
  }
  if (dtype != CHEB_F32 || n_iv < 1 || n_iv > kMaxResIntervals || covers != n_delta ||
      n_delta > residual_max_cover())
    return fail(CHEB_E_INVAL, "residual tables are malformed");
  for (int i = 0; i < n_iv; delta += iv[i].ncover, ++i)
    for (int64_t j = iv[i].vec_begin; j < iv[i].vec_begin + iv[i].n_vec; ++j)
      for (int e = 0; e < 4; ++e) {
        double sum = x_in ? double(x_in[4 * j + e]) : 0.0;
        for (int c = 0; c < iv[i].ncover; ++c)
          for (int k = 0; k < n; ++k) {
            const int64_t v = delta[c] + j;
            const uint64_t at =
                base[k] + 16u * uint64_t(v / kChunkVecs * super_vecs + v % kChunkVecs);
            sum += w[k] * double(reinterpret_cast<const float *>(at)[e]);
          }
        x_out[4 * j + e] = float(sum);
      }
  g_residual_launches.fetch_add(1);
  return ok();
}

int launch_residual(int dtype, int n, const uint64_t *base, const double *w, const int64_t *delta,
                    int ncover, const float *x_in, float *x_out, int64_t vec_begin,
                    int64_t n_vec, int64_t super_vecs, hipStream_t stream) {
  const ResidualInterval iv{vec_begin, n_vec, ncover};
  return launch_residual_intervals(dtype, n, base, w, delta, ncover, &iv, 1, x_in, x_out,
                                   super_vecs, stream);
}

}  // namespace cheb
