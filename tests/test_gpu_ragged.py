"""Channel counts that are multiples of 4 but of nothing larger: the staging modes that clear the channels past the last one,
and the store paths of pixel rows that are not 16-byte aligned."""
import numpy as np
import pytest
import torch

from paper_2411_00288_amd import workloads as wl
from helpers import check_close, dev_bits, layer_desc, oracle_ref, run_gpu
import oracle

pytestmark = pytest.mark.gpu


def L_(N, H, W, cin, cout, k, s=1, p=0, dtype=wl.F16, act=wl.ACT_RELU, seed=11):
    return wl.Layer(f"n{N}h{H}w{W}c{cin}o{cout}k{k}s{s}d{dtype}", N=N, H=H, W=W, cin=cin, cout=cout, kh=k, kw=k, stride=s, pad=p,
                    dtype=dtype, act=act, mask="logits", seed=seed)


SHAPES = [
    L_(2, 9, 7, 12, 38, 3, p=1), L_(1, 6, 11, 36, 70, 3, s=2, p=1, dtype=wl.BF16), L_(2, 7, 9, 80, 136, 3, p=1),
    L_(1, 5, 5, 40, 20, 3, p=1, dtype=wl.BF16), L_(2, 8, 10, 20, 66, 2, s=2), L_(1, 9, 9, 100, 260, 2, s=2, dtype=wl.BF16),
    L_(3, 7, 7, 76, 33, 1), L_(2, 5, 13, 132, 130, 1, dtype=wl.BF16), L_(1, 4, 5, 12, 10, 1),
]


@pytest.mark.parametrize("sparse", [True, False])
@pytest.mark.parametrize("tile", [None, 0, 1, 2, 3, 4, 5])
@pytest.mark.parametrize("L", SHAPES, ids=lambda L: L.name)
def test_ragged_channels_match_oracle(ss, force_tile, L, tile, sparse):
    d = wl.make_inputs(L)
    force_tile(tile)
    check_close(run_gpu(ss, L, d, sparse=sparse), oracle_ref(L, d), L.name)


@pytest.mark.parametrize("cout", [38, 33, 44])
def test_ragged_rows_with_a_residual(ss, cout):
    L = L_(2, 6, 7, 28, cout, 3, p=1, dtype=wl.BF16)
    d = wl.make_inputs(L)
    res = wl.to_bits(np.random.Generator(np.random.PCG64(3)).standard_normal((L.N, L.Ho, L.Wo, cout), dtype=np.float32), L.dtype)
    desc = layer_desc(ss, L)
    packed = ss.ss_mask_compress(desc, dev_bits(d["W"], L.dtype), torch.from_numpy(d["M"]).cuda())
    y = ss.ss_conv2d_res_fwd(desc, dev_bits(d["x"], L.dtype), packed, torch.from_numpy(d["bias"]).cuda(), dev_bits(res, L.dtype), (1, 1),
                             (1, 1), L.act)
    ref = oracle.conv2d(d["x"], d["W"], d["M"], cin=L.cin, kh=3, kw=3, korder=L.korder, dtype=L.dtype, bias=d["bias"], stride=(1, 1),
                        pad=(1, 1), act=L.act, residual=res)
    check_close(y, ref, L.name)


@pytest.mark.parametrize("k,s", [(1, 1), (2, 2)])
def test_channels_of_the_next_pixel_do_not_leak(ss, k, s):
    """Windows that do not overlap: a NaN pixel reaches its own output only (cin % 8 == 4, first and last pixel included)."""
    L = L_(1, 4, 6, 76, 40, k, s=s)
    d = wl.make_inputs(L)
    desc = layer_desc(ss, L)
    packed = ss.ss_mask_compress(desc, dev_bits(d["W"], L.dtype), torch.from_numpy(d["M"]).cuda())
    for px in [(0, 0), (1, 3), (3, 5)]:
        x = dev_bits(d["x"], L.dtype).clone()
        x[0, px[0], px[1]] = float("nan")
        bad = torch.isnan(ss.ss_conv2d_fwd(desc, x, packed, None, (s, s))).any(dim=3)[0].cpu()
        want = torch.zeros_like(bad)
        want[px[0] // s, px[1] // s] = True
        assert torch.equal(bad, want)
