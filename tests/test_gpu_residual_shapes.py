"""The residual kernel's launch shapes: tiles of 64 vectors shared by 1, 2, 4 or
16 waves, blocks of 16 tiles with a wave each, several residual intervals in
one launch, and tiles that cross the chunks of an interleaved entry, against
the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_23429_amd as cheb
from tests.gpu_util import say, to_host_bits

pytestmark = pytest.mark.gpu

DT = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}
# fp64 accumulation of at most (n * segments + 1) terms and one fp32 rounding:
# 2^-24 |o|, with the fp64 terms below 2^-40 of the floor (10^-3 S).
RES_TOL = 1e-6


def _check(dtype, n, seg_numel, res_off, res_n, layout, with_x, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    cache = cheb.ChebCache(n, DT[dtype], seg_numel, layout=layout)
    entries = []
    for k in range(n):
        segs = [torch.randn(s, generator=g, device="cuda").to(DT[dtype]) for s in seg_numel]
        cache.push(float(k), segs)
        entries.append(segs)
    w = np.random.default_rng(seed).standard_normal(n)
    x_in = torch.randn(res_n, generator=g, device="cuda") if with_x else None
    x_out = torch.full((res_n,), float("nan"), device="cuda")
    say(f"residual shape {dtype} n={n} segs={len(seg_numel)} res={res_n} {layout} x={with_x}")
    cache.residual_apply(w, res_off, x_out, x_in)
    torch.cuda.synchronize()
    # the entries as the cache lays them out: each segment from its offset
    hosts = []
    for segs in entries:
        flat = np.zeros(cache.slot_numel, dtype=np.float32 if dtype == "f32" else np.uint16)
        for o, s in zip(cache.seg_offset, segs):
            flat[o:o + s.numel()] = to_host_bits(s)
        hosts.append(flat)
    exp, mag = oracle.residual(hosts, w, cache.seg_offset, cache.seg_numel, res_off, res_n,
                               x_in=None if x_in is None else x_in.cpu().numpy(), dtype=dtype)
    e = oracle.parity_error(x_out.cpu().numpy().astype(np.float64), exp, mag)[0]
    assert e <= RES_TOL, e
    cache.close()


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("n", [1, 2, 3, 7])
@pytest.mark.parametrize("ncover", [1, 2, 3, 4, 5, 16, 17, 31])
def test_small_residual(dtype, n, ncover):
    """One tile and a bit: 1, 4 and 16 waves, partial groups of segments."""
    vec = 4 if dtype == "f32" else 8
    _check(dtype, n, [65 * vec] * ncover, [0] * ncover, 65 * vec, "slots", ncover % 2 == 0, ncover)


@pytest.mark.parametrize("layout", ["slots", "interleaved"])
@pytest.mark.parametrize("n,ncover,vecs", [(4, 1, 32 * 64 * 256 + 1), (1, 2, 64 * 64 * 256 + 1), (2, 3, 64 * 64 * 256 + 63),
                                           (7, 5, 16 * 64 * 256 + 1), (6, 24, 16 * 64 * 256 + 2),
                                           (2, 9, 16 * 64 * 256 + 65), (3, 6, 64 * 300 + 31),
                                           (3, 5, 4 * 64 * 256 + 7), (3, 5, 8 * 64 * 256 + 7),
                                           (2, 33, 32 * 64 * 256 + 9), (1, 24, 32 * 64 * 256 + 1),
                                           (1, 5, 32 * 64 * 256 + 1)])
def test_many_tiles(layout, n, ncover, vecs):
    """Residuals past each size at which the rule changes; odd vector counts
    put later segments' tiles across chunk ends."""
    _check("bf16", n, [vecs * 8] * ncover, [0] * ncover, vecs * 8, layout, True, ncover)


@pytest.mark.parametrize("layout", ["slots", "interleaved"])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n,ncover,tiles", [(4, 5, 13), (3, 3, 13), (8, 7, 14), (2, 9, 15),
                                            (1, 3, 5), (1, 2, 40), (1, 13, 28), (3, 5, 28),
                                            (5, 6, 40), (8, 3, 33)])
def test_blocks_of_tiles(layout, dtype, n, ncover, tiles):
    """Blocks of 16 tiles (single runs and pairs), the last block partly idle
    and the last tile partly filled; two intervals, so that a block holds tiles
    of both; numbers of segments that the loads of 2 or 4 do not divide."""
    vec = 4 if dtype == "f32" else 8
    vecs = tiles * 64 * 256 - 64 * 5 - 31
    head = 64 * 37 + 5                          # the first segments cover only this
    _check(dtype, n, [vecs * vec] * ncover, [0] * ncover, vecs * vec, layout, ncover % 2 == 1, n)
    _check(dtype, n, [head * vec] * 2 + [vecs * vec] * (ncover - 1), [0] * (ncover + 1),
           vecs * vec, layout, ncover % 2 == 0, n)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n", [1, 2, 5])
@pytest.mark.parametrize("extra", [0, 1, 63, 64, 65, 128, 4095, 4096, 4097, 8191])
def test_pairs_of_runs(dtype, n, extra):
    """Contiguous entries in pairs of runs 4096 vectors apart: whole pairs of
    4096 and every kind of rest behind them (none, one run, odd, one vector
    short of whole)."""
    vec = 4 if dtype == "f32" else 8
    vecs = 26 * 8192 + extra                   # over 12 tiles a compute unit
    _check(dtype, n, [vecs * vec] * 5, [0] * 5, vecs * vec, "slots", extra % 2 == 0, extra)


@pytest.mark.parametrize("layout", ["slots", "interleaved"])
@pytest.mark.parametrize("n_intervals", [2, 8, 9])
def test_intervals(layout, n_intervals):
    """Several intervals in one launch (up to 8) or in launches of their own
    (9), one of them covered by no segment, segments crossing chunk ends."""
    unit = 8 * 777
    res_n = unit * n_intervals
    seg, off = [], []
    for i in range(n_intervals):
        if i == 1:
            continue                           # nothing adds here
        for _ in range(1 + i % 3):
            seg.append(unit)
            off.append(unit * i)
    for x in (True, False):
        _check("bf16", 3, seg, off, res_n, layout, x, n_intervals)


@pytest.mark.parametrize("layout", ["slots", "interleaved"])
@pytest.mark.parametrize("ncover", [1, 3, 5, 17])
def test_zeros_keep_their_sign(layout, ncover):
    """A sum that starts from the residual itself: elements that no segment
    covers come out bit for bit (both zeros, infinities, subnormals), and a
    negative zero plus terms of negative zero stays one.  Exact."""
    half = 8 * 65
    x_in = torch.tensor([-0.0, 0.0, 1e-42, -1e-42, float("inf"), -float("inf"), -3.5, 7.25],
                        device="cuda").repeat(2 * half // 8)
    x_in[:half] = -0.0
    cache = cheb.ChebCache(2, torch.bfloat16, [half] * ncover, layout=layout)
    for k in range(2):
        cache.push(float(k), [torch.full((half,), -0.0, dtype=torch.bfloat16, device="cuda")] *
                   ncover)
    say(f"residual zeros {layout} segs={ncover}")
    for x in (x_in, None):
        out = cache.residual_apply([0.5, 2.0], [0] * ncover, torch.empty_like(x_in), x)
        want = torch.zeros_like(x_in) if x is None else x_in
        assert torch.equal(out.view(torch.int32), want.view(torch.int32))
    cache.close()
