"""The push's 64-vector tiles: segments around a tile's end, ragged and empty
ones, very unlike sizes (in classes of like size, largest first), equal ones that
start anywhere in a tile, and more segments than one launch takes, read back
bit for bit with zeroed padding."""
import pytest
import torch

import paper_2608_23429_amd as cheb
from tests.gpu_util import say

pytestmark = pytest.mark.gpu

DT = {"bf16": torch.bfloat16, "f32": torch.float32}
SIZES = {
    "tile_edges": [1, 7, 8, 9, 511, 512, 513, 519, 520, 521, 1023, 1024, 1025],
    "empty": [0, 512, 0, 3, 0],
    "unlike": [5, 16385 * 512, 3, 16385 * 512 + 9, 700, 16000 * 512, 8],
    "alike_shifted": [528] * 70,               # tiles per segment vary with its place
    "many": [(j * 37) % 2000 for j in range(150)],
    "all_unlike": [int(500 * 1.25 ** j) for j in range(35)],   # more sizes than classes
}


@pytest.mark.parametrize("layout", ["slots", "interleaved"])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("sizes", sorted(SIZES))
def test_push_reads_back(layout, dtype, sizes):
    seg = SIZES[sizes]
    cache = cheb.ChebCache(3, DT[dtype], seg, layout=layout)
    cache.arena.fill_(0xA5)
    g = torch.Generator(device="cuda")
    g.manual_seed(len(seg))
    want = []
    for k in range(4):                         # the fourth evicts the first
        flat = torch.zeros(cache.slot_numel, dtype=DT[dtype], device="cuda")
        src = [torch.randn(n, generator=g, device="cuda").to(DT[dtype]) for n in seg]
        for o, s in zip(cache.seg_offset, src):
            flat[o:o + s.numel()] = s
        say(f"push {sizes} {dtype} {layout} {k}")
        cache.push(float(k), src)
        want.append(flat)
    torch.cuda.synchronize()
    for k in range(3):
        got = cache.entry(k)
        assert torch.equal(got.view(torch.uint8), want[k + 1].view(torch.uint8)), k
    cache.close()
