"""The resident inverted bottleneck (tile id 42: a wave takes 32 pixels through both layers, weights in LDS) against the one-tile kernel (id 40), whose sums
it forms in the same order: bit for bit, with pixel tails around a tile, fewer and more tiles than waves, the shortest and the longest
intermediates that fit, and every option of the call.  The one-tile kernel is compared with the oracle elsewhere."""
import numpy as np
import pytest
import torch

from paper_2411_00288_amd import workloads as wl
from test_gpu_fused import _pair, _run

pytestmark = pytest.mark.gpu

# pixels, channels, intermediate channels, workgroups at most (0: one per compute unit)
SHAPES = [(1, 96, 128, 0), (31, 96, 384, 0), (33, 128, 128, 0), (12 * 32 + 1, 96, 384, 1), (25 * 32 + 17, 96, 256, 1), (8 * 32, 128, 512, 1),
          (17 * 32 + 5, 128, 512, 2), (1000, 96, 640, 1), (9000, 96, 384, 0)]


@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_equals_the_one_tile_kernel(ss, force_tile, shape):
    P, C, cmid, limit = shape
    i = SHAPES.index(shape)
    res = np.random.default_rng(i).standard_normal((1, 1, P, C), dtype=np.float32)
    for dtype, act1, act2, with_res in ((wl.BF16, wl.ACT_GELU, wl.ACT_NONE, True), (wl.BF16, wl.ACT_RELU, wl.ACT_NONE, True), (wl.F16, (wl.ACT_RELU, wl.ACT_NONE)[i % 2], (wl.ACT_RELU, wl.ACT_GELU)[i % 2], i % 3 == 0)):
        L1, L2 = _pair(1, 1, P, C, cmid, C, k=1, p=0, dtype=dtype, act1=act1, act2=act2, seed=70 + i)
        d1, d2 = wl.make_inputs(L1), wl.make_inputs(L2)
        bits = wl.to_bits(res, dtype) if with_res else None
        for sparse in (True, False):
            # (what the resident kernel cannot run: forced or not, the one-tile kernel does)
            if (sparse and act1 == wl.ACT_GELU) or (not sparse and (C == 128 or cmid > 384)):
                continue
            force_tile(40)
            expect = _run(ss, L1, L2, d1, d2, bits, sparse)[0]
            force_tile(42)
            ss.ss_debug_limit_blocks(limit)
            try:
                got = _run(ss, L1, L2, d1, d2, bits, sparse)[0]
            finally:
                ss.ss_debug_limit_blocks(0)
            assert torch.isfinite(got).all() and torch.equal(got.view(torch.int16), expect.view(torch.int16)), (shape, dtype, sparse)


def test_non_finite_values_stay_with_their_pixel(ss, force_tile):
    """A NaN and an infinity in the input and in the residual reach what they reach in the one-tile kernel and nothing else."""
    P, C = 100, 96
    L1, L2 = _pair(1, 1, P, C, 4 * C, C, k=1, p=0, act1=wl.ACT_NONE, act2=wl.ACT_NONE, seed=90)
    d1, d2 = wl.make_inputs(L1), wl.make_inputs(L2)
    r = np.random.default_rng(3).standard_normal((1, 1, P, C), dtype=np.float32)
    r[0, 0, 40, 7], r[0, 0, 41, 50] = np.nan, np.inf
    res = wl.to_bits(r, L1.dtype)
    d1["x"] = d1["x"].copy()
    d1["x"].reshape(P, C)[70, 3] = wl.to_bits(np.full(1, np.nan, np.float32), L1.dtype)[0]
    out = {}
    for tile in (40, 42):
        force_tile(tile)
        out[tile] = _run(ss, L1, L2, d1, d2, res, True)[0].float().reshape(P, C).cpu()
    assert torch.equal(torch.isnan(out[40]), torch.isnan(out[42])) and torch.equal(out[40].nan_to_num(), out[42].nan_to_num())
    bad = ~torch.isfinite(out[42])
    assert bad[70].all() and bad.sum().item() == C + 2 and bad[40, 7] and bad[41, 50]
