"""The depthwise kernels that the library chooses by the number of outputs, each forced (tile ids 60 to 65: vector ALU, matrix unit, few outputs with 1 x 2, 1 x 4,
2 x 4 and 4 x 4 outputs per thread): images smaller than a thread's outputs, one past them, paddings from none to more than the filter, against
the oracle; a non-finite value stays in its window."""
import numpy as np
import pytest
import torch

import oracle
from helpers import check_close, host_bits
from paper_2411_00288_amd import workloads as wl
from test_gpu_dwconv import _run

pytestmark = pytest.mark.gpu

KINDS = [(k, t) for k, ids in ((3, (60, 63, 64, 65)), (5, (60, 61, 63)), (7, (60, 61, 62, 63, 64))) for t in ids]
SHAPES = [(1, 1, 1, 8), (2, 3, 17, 40), (1, 20, 33, 16), (3, 5, 9, 104), (9, 6, 8, 32), (2, 13, 4, 160)]


@pytest.mark.parametrize("k,tile", KINDS)
def test_against_oracle(ss, force_tile, k, tile):
    force_tile(tile)
    for i, (N, H, W, C) in enumerate(SHAPES):
        dtype, act = (wl.BF16, wl.F16)[i % 2], (wl.ACT_NONE, wl.ACT_RELU)[i // 2 % 2]
        rng = np.random.Generator(np.random.PCG64(10 * k + i))
        xb = wl.to_bits(rng.standard_normal((N, H, W, C), dtype=np.float32), dtype)
        wb = wl.to_bits(rng.standard_normal((k, k, C), dtype=np.float32) * np.float32((2.0 / (k * k)) ** 0.5), dtype)
        bias = None if i == 3 else (rng.standard_normal(C) * 0.1).astype(np.float32)
        for p in (k // 2, k // 2 + 2, 0):
            if H + 2 * p < k or W + 2 * p < k:
                continue
            ref = oracle.dwconv2d(xb, wb, dtype=dtype, bias=bias, pad=(p, p), act=act)
            check_close(_run(ss, xb, wb, bias, dtype, (p, p), act), ref, f"{(N, H, W, C)} k {k} pad {p} tile {tile}")


@pytest.mark.parametrize("k,tile", KINDS)
def test_non_finite_values_stay_in_their_windows(ss, force_tile, k, tile):
    force_tile(tile)
    x = torch.randn((2, 12, 14, 16), device="cuda").to(torch.bfloat16)
    w = torch.rand((k, k, 16), device="cuda").to(torch.bfloat16) + 0.5
    h = k // 2
    clean = ss.ss_dwconv2d_fwd(x, w, None, (h, h))
    for value in (float("nan"), float("inf")):
        z = x.clone()
        z[1, 0, 13, 5] = value                            # a corner: the next row, the next image's first row and the columns behind it must not see it
        y = ss.ss_dwconv2d_fwd(z, w, None, (h, h))
        hit = torch.zeros(y.shape, dtype=torch.bool, device="cuda")
        hit[1, :h + 1, 13 - h:, 5] = True
        assert not torch.isfinite(y[hit].float()).any()
        assert torch.equal(y[~hit].view(torch.int16), clean[~hit].view(torch.int16)) or tile == 61
        assert torch.isfinite(y[~hit].float()).all()


def test_sizes_where_the_choice_changes(ss, force_tile):
    """On either side of each line the library's result is, bit for bit, that of the kernel named for that side."""
    ncu = torch.cuda.get_device_properties(0).multi_processor_count
    pairs = 256 * ncu // (7 * 48)                         # rows of 14 columns and 96 channels that make one workgroup per unit in pairs of columns
    for k, (N, H, W, C), tile in ((3, (1, 500, 49, 96), 63), (3, (1, 560, 50, 96), 64), (3, (1, 1700, 50, 96), 65), (5, (1, 1040, 50, 96), 63),
                                  (5, (1, 1050, 50, 96), 61), (7, (1, pairs, 14, 96), 62), (7, (1, pairs + 1, 14, 96), 63), (7, (1, 350, 50, 96), 63),
                                  (7, (1, 360, 50, 96), 64), (7, (1, 660, 50, 96), 64), (7, (1, 670, 50, 96), 61)):
        x = torch.randn((N, H, W, C), device="cuda").to(torch.bfloat16)
        w = (torch.randn((k, k, C), device="cuda") / k).to(torch.bfloat16)
        force_tile(None)
        y = ss.ss_dwconv2d_fwd(x, w, None, (k // 2, k // 2))
        force_tile(tile)
        z = ss.ss_dwconv2d_fwd(x, w, None, (k // 2, k // 2))
        assert torch.equal(y.view(torch.int16), z.view(torch.int16)), (k, N, H, W, C)
        ref = oracle.dwconv2d(host_bits(x[:, :16]), host_bits(w), dtype=wl.BF16, pad=(k // 2, k // 2))
        check_close(y[:, :16 - k // 2], ref[:, :16 - k // 2], f"{(N, H, W, C)} k {k}")
