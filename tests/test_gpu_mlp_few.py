"""The inverted bottleneck on few pixels (tile id 41: a wave for each 32 intermediate channels) against the oracle chain, beside the kernel it stands in
for (id 40): every number of waves, output row tiles that do and do not divide it, shares of the reduction that are empty, pixel tails around a
workgroup's 32, both sides of the line between the two kernels."""
import numpy as np
import pytest
import torch

from paper_2411_00288_amd import workloads as wl
from test_gpu_fused import _oracle_pair, _pair, _run

pytestmark = pytest.mark.gpu

# pixels, input, intermediate and output channels
SHAPES = [(1, 32, 128, 32), (31, 64, 128, 96), (32, 96, 256, 96), (33, 128, 256, 32), (65, 32, 384, 128), (50, 96, 384, 64), (40, 128, 512, 96),
          (64, 64, 512, 32), (97, 128, 512, 128)]


@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("tile", [40, 41])
def test_against_oracle(ss, force_tile, tile, shape):
    P, cin, cmid, cout = shape
    i = SHAPES.index(shape)
    force_tile(tile)
    for dtype, act1, act2, with_res in ((wl.BF16, wl.ACT_GELU, wl.ACT_NONE, True), (wl.F16, wl.ACT_RELU, (wl.ACT_GELU, wl.ACT_RELU)[i % 2], i % 3 == 0)):
        L1, L2 = _pair(1, 1, P, cin, cmid, cout, k=1, p=0, dtype=dtype, act1=act1, act2=act2, seed=40 + i)
        d1, d2 = wl.make_inputs(L1), wl.make_inputs(L2)
        rng = np.random.Generator(np.random.PCG64(i))
        res = wl.to_bits(rng.standard_normal((1, 1, P, cout), dtype=np.float32), dtype) if with_res else None
        _t, ref = _oracle_pair(L1, L2, d1, d2, res)
        for sparse in (True, False):
            y, _sep, _t = _run(ss, L1, L2, d1, d2, res, sparse)
            got, what = y.float().cpu().numpy().astype(np.float64), f"{shape} tile {tile} dtype {dtype} sparse {sparse}"
            # (two layers' roundings, as in test_fused_pair_matches_oracle_chain)
            assert np.isfinite(got).all() and np.linalg.norm(got - ref) <= 4e-3 * np.linalg.norm(ref), what
            assert (np.abs(got - ref) <= 2e-2 * (np.abs(ref) + 1)).all(), what


def test_both_sides_of_the_line(ss, force_tile):
    """One workgroup of 32 pixels per compute unit, and one more: the two kernels differ in the order of fp32 sums only, and the library's own
    choice equals one of them bit for bit.  The output may take the residual's place."""
    ncu = torch.cuda.get_device_properties(0).multi_processor_count
    for P in (32 * ncu, 32 * ncu + 1):
        L1, L2 = _pair(1, 1, P, 64, 256, 64, k=1, p=0, act1=wl.ACT_GELU, act2=wl.ACT_NONE, seed=60)
        d1, d2 = wl.make_inputs(L1), wl.make_inputs(L2)
        res = wl.to_bits(np.random.default_rng(1).standard_normal((1, 1, P, 64)).astype(np.float32), L1.dtype)
        out = {}
        for tile in (None, 40, 41):
            force_tile(tile)
            out[tile] = _run(ss, L1, L2, d1, d2, res, True)[0]
        a, b = out[40].double(), out[41].double()
        assert (torch.linalg.norm(a - b) <= 2e-3 * torch.linalg.norm(a)).item()
        assert torch.equal(out[None].view(torch.int16), out[41 if P == 32 * ncu else 40].view(torch.int16))
