// How a residual call is cut into launches, on the CPU: the library's host
// sources are linked against tests/host_stubs.cpp, whose residual launcher
// checks the tables it is given and adds fp32 entries in host memory as they
// say.  Random segment maps (gaps, overlaps, up to 8 intervals in one launch
// and more in launches of their own, more segments over one element than a
// table holds) in both layouts, with, without and in place of a residual,
// against the plain sum over the segments.  Pushes of random layouts, from like
// sizes to all different ones, go through the stub's check of their launches.
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>

#include <random>
#include <vector>

#include "internal.h"

extern "C" void stub_gather_batches_ok(int n);
extern "C" void stub_residual_on_host(int on);
extern "C" int stub_residual_launches();

#define CHECK(cond)                                                                      \
  do {                                                                                   \
    if (!(cond)) {                                                                       \
      fprintf(stderr, "line %d, seed %d: %s (%s)\n", __LINE__, g_seed, #cond,            \
              cheb_last_error());                                                        \
      exit(1);                                                                           \
    }                                                                                    \
  } while (0)

static int g_seed = 0;

static void one(int seed) {
  g_seed = seed;
  std::mt19937 rng(seed);
  auto pick = [&](int lo, int hi) { return lo + int(rng() % uint32_t(hi - lo + 1)); };
  const int layout = seed % 2 ? CHEB_LAYOUT_INTERLEAVED : CHEB_LAYOUT_SLOTS;
  const int n = pick(1, 4), unit = 4 * pick(1, 400), parts = pick(1, 11);
  const int64_t res_numel = int64_t(unit) * parts;
  std::vector<int64_t> numel, off;
  const int segs = seed % 7 == 0 ? 300 : pick(1, 40);
  for (int s = 0; s < segs; ++s) {
    const int first = pick(0, parts - 1), last = seed % 3 ? first : pick(first, parts - 1);
    numel.push_back(pick(0, 19) ? int64_t(unit) * (last - first + 1) : 0);
    off.push_back(pick(0, 9) ? int64_t(unit) * first : -1);
  }
  size_t bytes = 0;
  CHECK(cheb_cache_arena_bytes_ex(n, CHEB_F32, numel.data(), segs, layout, &bytes) == CHEB_OK);
  if (bytes == 0) return;
  char *arena = static_cast<char *>(aligned_alloc(256, (bytes + 255) / 256 * 256));
  cheb_cache *c = nullptr;
  CHECK(cheb_cache_create_ex(&c, n, CHEB_F32, numel.data(), segs, layout, arena, bytes) ==
        CHEB_OK);
  // The stub's copies do nothing; the entries are filled by the chunk formula.
  std::vector<const void *> src(segs, arena);
  for (int k = 0; k < n; ++k) CHECK(cheb_cache_push(c, k, src.data(), nullptr) == CHEB_OK);
  int64_t slot_numel = 0, chunk = 0, stride = 0;
  int32_t lay = 0;
  CHECK(cheb_cache_slot_numel(c, &slot_numel) == CHEB_OK);
  CHECK(cheb_cache_geometry(c, &lay, &chunk, &stride) == CHEB_OK);
  std::vector<std::vector<float>> entry(n, std::vector<float>(size_t(slot_numel)));
  std::vector<double> w(n);
  for (int k = 0; k < n; ++k) {
    w[k] = 0.25 * pick(-8, 8);
    void *base = nullptr;
    CHECK(cheb_cache_entry(c, k, &base) == CHEB_OK);
    for (int64_t i = 0; i < slot_numel; ++i) {
      entry[k][i] = float(pick(-1000, 1000));      // sums stay exact
      const int64_t at = lay == CHEB_LAYOUT_SLOTS ? i : i / chunk * stride + i % chunk;
      static_cast<float *>(base)[at] = entry[k][i];
    }
  }
  float *x_in = static_cast<float *>(aligned_alloc(16, size_t(res_numel) * 4));
  float *x_out = static_cast<float *>(aligned_alloc(16, size_t(res_numel) * 4));
  std::vector<double> want(res_numel), reduced(res_numel);
  for (int64_t j = 0; j < res_numel; ++j) {
    x_in[j] = float(pick(-1000, 1000));
    x_out[j] = -1e30f;
  }
  for (int s = 0; s < segs; ++s) {
    if (off[s] < 0) continue;
    int64_t at = 0;
    CHECK(cheb_cache_segment_offset(c, s, &at) == CHEB_OK);
    for (int64_t i = 0; i < numel[s]; ++i)
      for (int k = 0; k < n; ++k) {
        want[off[s] + i] += w[k] * entry[k][at + i];
        if (k == 0) reduced[off[s] + i] += entry[0][at + i];
      }
  }
  auto same = [&](const std::vector<double> &sum, const float *x) {
    for (int64_t j = 0; j < res_numel; ++j) CHECK(x_out[j] == float((x ? x[j] : 0.0) + sum[j]));
  };
  const std::vector<float> x0(x_in, x_in + res_numel);
  CHECK(cheb_residual_apply(c, w.data(), off.data(), res_numel, x_in, x_out, nullptr) == CHEB_OK);
  same(want, x_in);
  CHECK(cheb_residual_apply(c, w.data(), off.data(), res_numel, nullptr, x_out, nullptr) ==
        CHEB_OK);
  same(want, nullptr);
  for (int64_t j = 0; j < res_numel; ++j) x_out[j] = x0[j];
  CHECK(cheb_residual_apply(c, w.data(), off.data(), res_numel, x_out, x_out, nullptr) == CHEB_OK);
  same(want, x0.data());
  // A full step's module outputs, each in memory of its own.
  std::vector<float *> own(segs);
  std::vector<const void *> outs(segs);
  for (int s = 0; s < segs; ++s) {
    int64_t at = 0;
    CHECK(cheb_cache_segment_offset(c, s, &at) == CHEB_OK);
    own[s] = static_cast<float *>(aligned_alloc(16, size_t(numel[s]) * 4 + 16));
    for (int64_t i = 0; i < numel[s]; ++i) own[s][i] = entry[0][at + i];
    outs[s] = own[s];
  }
  CHECK(cheb_residual_reduce(outs.data(), numel.data(), off.data(), segs, CHEB_F32, x_in, x_out,
                             res_numel, nullptr) == CHEB_OK);
  same(reduced, x_in);
  for (float *p : own) free(p);
  free(x_in);
  free(x_out);
  CHECK(cheb_cache_destroy(c) == CHEB_OK);
  free(arena);
}

// The arena is never dereferenced.
static void pushes(int seed) {
  g_seed = seed;
  std::mt19937_64 rng(uint64_t(seed) + 1000);
  const int layout = seed % 2 ? CHEB_LAYOUT_INTERLEAVED : CHEB_LAYOUT_SLOTS;
  const int dtype = int(rng() % 3), segs = 1 + int(rng() % 200), kinds = 1 + int(rng() % 40);
  std::vector<int64_t> size(kinds), numel(segs);
  for (int64_t &n : size) n = int64_t(rng() >> (38 + rng() % 26));  // to 2^26
  for (int64_t &n : numel) n = size[rng() % size.size()];
  size_t bytes = 0;
  if (cheb_cache_arena_bytes_ex(2, dtype, numel.data(), segs, layout, &bytes) != CHEB_OK) return;
  void *arena = reinterpret_cast<void *>(uintptr_t(1) << 44);
  cheb_cache *c = nullptr;
  if (bytes == 0) return;
  CHECK(cheb_cache_create_ex(&c, 2, dtype, numel.data(), segs, layout, arena, bytes) == CHEB_OK);
  std::vector<const void *> src(segs, arena);
  CHECK(cheb_cache_push(c, 1.0, src.data(), nullptr) == CHEB_OK);
  CHECK(cheb_cache_destroy(c) == CHEB_OK);
}

int main() {
  stub_residual_on_host(1);
  stub_gather_batches_ok(1 << 30);
  for (int seed = 0; seed < 300; ++seed) one(seed);
  for (int seed = 0; seed < 3000; ++seed) pushes(seed);
  // Image and text tokens: two intervals, one launch.
  const int64_t numel[] = {64, 16, 80}, off[] = {16, 0, 0};
  alignas(16) static float buf[160], x[80];
  const void *src[] = {buf, buf + 64, buf + 80};
  const int before = stub_residual_launches();
  CHECK(cheb_residual_reduce(src, numel, off, 3, CHEB_F32, nullptr, x, 80, nullptr) == CHEB_OK);
  CHECK(stub_residual_launches() == before + 1);
  printf("residual plan ok\n");
  return 0;
}
