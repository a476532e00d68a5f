"""The prediction's one-wave tiles at their edges: vector counts around the
64-vector tile and the 2048-vector chunk, ragged tails, both layouts and one
or several outputs, against the oracle and bit for bit against the
256-lane launch shape."""
import numpy as np
import pytest
import torch

import oracle
import paper_2608_23429_amd as cheb
from tests.gpu_util import check_parity, say, to_host_bits

pytestmark = pytest.mark.gpu

DT = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}
VECS = [0, 1, 63, 64, 65, 127, 128, 2047, 2048, 2049, 4096 + 64]


@pytest.fixture(autouse=True)
def default_shape():
    yield
    cheb.cheb_set_launch_config(**cheb.DEFAULT_LAUNCH_CONFIG)


def _same(a, b):
    return torch.equal(a.view(torch.uint8), b.view(torch.uint8))


@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("n,m", [(1, 1), (3, 2), (6, 1), (8, 5)])
def test_stateless_tiles(dtype, n, m):
    vec = 4 if dtype == "f32" else 8
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    # targets at most 0.4 past n - 0.5: sum |w| is below 200 at n = 8,
    # so no result of normal values (below 6 each) leaves binary16's range (a target
    # 4 ahead would: sum |w| is 38455 there)
    w = np.stack([oracle.weights_row(np.arange(n, dtype=float), n - 0.5 + 0.1 * j)
                  for j in range(m)])
    for vecs in VECS:
        for tail in (0, 1, vec - 1):
            numel = vecs * vec + tail
            if numel == 0:
                continue
            srcs = [torch.randn(numel, generator=g, device="cuda").to(DT[dtype]) for _ in range(n)]
            outs = [torch.empty(numel, dtype=DT[dtype], device="cuda") for _ in range(m)]
            say(f"tiles {dtype} n={n} m={m} numel={numel}")
            cheb.combine_multi(srcs, w, outs)
            torch.cuda.synchronize()
            for j in range(m):
                check_parity(to_host_bits(outs[j]), [to_host_bits(s) for s in srcs], w[j], dtype)
            cheb.cheb_set_launch_config(block=256)
            for j in range(m):
                other = torch.empty_like(outs[j])
                cheb.combine(srcs, w[j], other)
                torch.cuda.synchronize()
                assert _same(other, outs[j])
            cheb.cheb_set_launch_config(**cheb.DEFAULT_LAUNCH_CONFIG)


@pytest.mark.parametrize("layout", ["slots", "interleaved"])
@pytest.mark.parametrize("n,m", [(2, 1), (3, 1), (5, 3)])
def test_ring_tiles(layout, n, m):
    """Sizes on both sides of the 512 KiB a compute unit at which the number
    of blocks in flight changes, and tiles at chunk ends."""
    w = np.stack([oracle.weights_row(np.arange(n, dtype=float), n + 0.25 * j) for j in range(m)])
    for vecs in (1, 65, 2048 + 1, 64 * 256 * 512 // (n + m) - 63, 64 * 256 * 512 // (n + m) + 65):
        numel = vecs * 8 - 3
        cache = cheb.ChebCache(n, torch.bfloat16, [numel], layout=layout)
        for k in range(n):
            cache.push(float(k), [torch.randn(numel, device="cuda").to(torch.bfloat16)])
        say(f"ring tiles {layout} n={n} m={m} vecs={vecs}")
        outs = cache.extrapolate_multi(w)
        torch.cuda.synchronize()
        hosts = [to_host_bits(cache.entry(k)) for k in range(n)]
        for j in range(m):
            check_parity(to_host_bits(outs[j]), hosts, w[j], "bf16")
        cheb.cheb_set_launch_config(block=256)
        for j in range(m):
            other = cache.extrapolate(w[j])
            torch.cuda.synchronize()
            assert _same(other, outs[j])
        cheb.cheb_set_launch_config(**cheb.DEFAULT_LAUNCH_CONFIG)
        cache.close()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("n,m", [(3, 1), (2, 2)])
@pytest.mark.parametrize("extra", [0, 1, 63, 64, 65, 4095, 4096, 4097, 8191])
def test_pairs_of_runs(dtype, n, m, extra):
    """Contiguous sources in pairs of runs 4096 vectors apart: whole pairs and
    every kind of rest behind them, with and without a ragged tail, bit for
    bit as the 256-lane shape gives it."""
    vec = 4 if dtype == "f32" else 8
    numel = (64 * 256 * 512 // (n + m) + extra) * vec + extra % vec
    g = torch.Generator(device="cuda")
    g.manual_seed(extra)
    srcs = [torch.randn(numel, generator=g, device="cuda").to(DT[dtype]) for _ in range(n)]
    w = np.stack([oracle.weights_row(np.arange(n, dtype=float), n + 0.5 * j) for j in range(m)])
    outs = [torch.full((numel,), float("nan"), dtype=DT[dtype], device="cuda") for _ in range(m)]
    say(f"pairs {dtype} n={n} m={m} numel={numel}")
    cheb.combine_multi(srcs, w, outs)
    cheb.cheb_set_launch_config(block=256)
    for j in range(m):
        other = torch.empty_like(outs[j])
        cheb.combine(srcs, w[j], other)
        torch.cuda.synchronize()
        assert _same(other, outs[j])
