"""GPU parity of the depthwise convolution against the fp64 oracle (ragged widths, every supported kernel width, both
dtypes), a bit-exact small-integer case, and the ConvNeXt-T stage-1 shape on sampled outputs."""
import numpy as np
import pytest
import torch

import oracle
from helpers import check_close, dev_bits, host_bits
from paper_2411_00288_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _run(ss, xb, wb, bias, dtype, pad, act):
    b = None if bias is None else torch.from_numpy(bias).cuda()
    y = ss.ss_dwconv2d_fwd(dev_bits(xb, dtype), dev_bits(wb, dtype), b, pad, act)
    torch.cuda.synchronize()
    return y


@pytest.mark.parametrize("shape", [(2, 9, 13, 24, 7, 7, 3), (3, 6, 7, 8, 3, 3, 1), (1, 11, 5, 40, 5, 5, 2), (2, 8, 9, 16, 3, 7, 0),
                                   (1, 7, 7, 96, 7, 7, 3), (1, 4, 3, 8, 3, 3, 2)])
@pytest.mark.parametrize("dtype", [wl.F16, wl.BF16])
def test_dwconv_matches_oracle(ss, shape, dtype):
    N, H, W, C, kh, kw, p = shape
    rng = np.random.Generator(np.random.PCG64(21))
    xb = wl.to_bits(rng.standard_normal((N, H, W, C), dtype=np.float32), dtype)
    wb = wl.to_bits(rng.standard_normal((kh, kw, C), dtype=np.float32) * np.float32((2.0 / (kh * kw)) ** 0.5), dtype)
    bias = (rng.standard_normal(C) * 0.1).astype(np.float32)
    for act in (wl.ACT_NONE, wl.ACT_RELU):
        ref = oracle.dwconv2d(xb, wb, dtype=dtype, bias=bias, pad=(p, p), act=act)
        check_close(_run(ss, xb, wb, bias, dtype, (p, p), act), ref, f"{shape} act {act}")
    ref = oracle.dwconv2d(xb, wb, dtype=dtype, bias=None, pad=(p, p))
    check_close(_run(ss, xb, wb, None, dtype, (p, p), wl.ACT_NONE), ref, f"{shape} no bias")


def test_dwconv_small_integers_are_bit_exact(ss):
    rng = np.random.Generator(np.random.PCG64(3))
    x = rng.integers(0, 3, size=(2, 10, 11, 16)).astype(np.float32)
    w = rng.integers(-1, 2, size=(7, 7, 16)).astype(np.float32)
    bias = rng.integers(-2, 3, size=16).astype(np.float32)
    for dtype in (wl.F16, wl.BF16):           # |sum| <= 2*49 + 2 = 100: exact in both types
        xb, wb = wl.to_bits(x, dtype), wl.to_bits(w, dtype)
        ref = oracle.dwconv2d(xb, wb, dtype=dtype, bias=bias, pad=(3, 3))
        y = _run(ss, xb, wb, bias, dtype, (3, 3), wl.ACT_NONE)
        assert np.array_equal(host_bits(y), wl.to_bits(ref.astype(np.float32), dtype))


def test_dwconv_convnext_stage1_shape_sampled(ss):
    N, H, W, C = 128, 56, 56, 96
    g = torch.Generator(device="cuda").manual_seed(1)
    x = torch.randn((N, H, W, C), generator=g, device="cuda").to(torch.bfloat16)
    w = (torch.randn((7, 7, C), generator=g, device="cuda") * (2.0 / 49) ** 0.5).to(torch.bfloat16)
    bias = torch.randn(C, generator=g, device="cuda") * 0.1
    y = ss.ss_dwconv2d_fwd(x, w, bias, (3, 3))
    torch.cuda.synchronize()
    # the oracle on a few whole images (first, middle, last) is cheap enough
    for n in (0, 61, 127):
        ref = oracle.dwconv2d(host_bits(x[n:n + 1]), host_bits(w), dtype=wl.BF16, bias=bias.cpu().numpy(), pad=(3, 3))
        check_close(y[n:n + 1], ref, f"image {n}")


def test_dwconv_argument_errors(ss):
    x = torch.zeros((1, 8, 8, 12), dtype=torch.float16, device="cuda")
    with pytest.raises(ss.SSError):
        ss.ss_dwconv2d_fwd(x, torch.zeros((3, 3, 12), dtype=torch.float16, device="cuda"))        # C % 8 != 0
    x = torch.zeros((1, 8, 8, 16), dtype=torch.float16, device="cuda")
    with pytest.raises(ss.SSError):
        ss.ss_dwconv2d_fwd(x, torch.zeros((3, 4, 16), dtype=torch.float16, device="cuda"))        # kernel width 4
    with pytest.raises(ss.SSError):
        ss.ss_dwconv2d_fwd(x, torch.zeros((3, 3, 16), dtype=torch.bfloat16, device="cuda"))       # dtype mismatch


@pytest.mark.parametrize("shape", [(1, 1, 1, 8, 7, 3), (2, 3, 17, 40, 7, 3), (1, 20, 33, 16, 7, 0), (3, 5, 70, 24, 7, 6), (9, 17, 8, 104, 7, 3),
                                   (70, 31, 30, 72, 5, 2)])
def test_matrix_kernel_edges(ss, shape):
    """Strips of 16 columns and several rows: images smaller than a strip, one column past it, channel groups half filled, more
    strips than workgroups walk in one go; without and with a large padding."""
    N, H, W, C, k, p = shape
    rng = np.random.Generator(np.random.PCG64(H * W))
    xb = wl.to_bits(rng.standard_normal((N, H, W, C), dtype=np.float32), wl.BF16)
    wb = wl.to_bits(rng.standard_normal((k, k, C), dtype=np.float32) * np.float32((2.0 / (k * k)) ** 0.5), wl.BF16)
    bias = (rng.standard_normal(C) * 0.1).astype(np.float32)
    y = _run(ss, xb, wb, bias, wl.BF16, (p, p), wl.ACT_RELU)
    check_close(y, oracle.dwconv2d(xb, wb, dtype=wl.BF16, bias=bias, pad=(p, p), act=wl.ACT_RELU), f"{shape}")


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_matrix_kernel_keeps_non_finite_values_in_their_windows(ss, value):
    x = torch.randn((1, 20, 40, 24), device="cuda").to(torch.bfloat16)
    w = torch.rand((7, 7, 24), device="cuda").to(torch.bfloat16) + 0.5
    clean = ss.ss_dwconv2d_fwd(x, w, None, (3, 3))
    x[0, 9, 14, 5] = value
    y = ss.ss_dwconv2d_fwd(x, w, None, (3, 3))
    hit = torch.zeros(y.shape, dtype=torch.bool, device="cuda")
    hit[0, 6:13, 11:18, 5] = True
    assert not torch.isfinite(y[hit].float()).any()
    assert torch.isfinite(y[~hit].float()).all()
    assert (y[~hit].float() - clean[~hit].float()).abs().max() <= 0.125      # (fp32 sums in another order, one rounding)


@pytest.mark.parametrize("shape", [(58, 19, 3, 520, 7), (58, 19, 9, 520, 5)])
def test_rows_dealt_out_evenly(ss, shape):
    """Four blocks of 16 images on seven workgroups of a channel group: runs of 10 or 11 of a block's 19 rows, some in two blocks; then a
    non-finite value, for which a workgroup goes through its runs again."""
    N, H, W, C, k = shape
    rng = np.random.Generator(np.random.PCG64(W))
    xb = wl.to_bits(rng.standard_normal((N, H, W, C), dtype=np.float32), wl.F16)
    wb = wl.to_bits(rng.standard_normal((k, k, C), dtype=np.float32) * np.float32((2.0 / (k * k)) ** 0.5), wl.F16)
    bias = (rng.standard_normal(C) * 0.1).astype(np.float32)
    y = _run(ss, xb, wb, bias, wl.F16, (k // 2, k // 2), wl.ACT_NONE)
    check_close(y, oracle.dwconv2d(xb, wb, dtype=wl.F16, bias=bias, pad=(k // 2, k // 2), act=wl.ACT_NONE), f"{shape}")
    xb[33, 10, 1, 77] = 0x7C00
    z = _run(ss, xb, wb, bias, wl.F16, (k // 2, k // 2), wl.ACT_NONE)
    hit = torch.zeros(z.shape, dtype=torch.bool, device="cuda")
    hit[33, 10 - k // 2:11 + k // 2, :2 + k // 2, 77] = True
    assert not torch.isfinite(z[hit].float()).any() and torch.isfinite(z[~hit].float()).all()
    assert (z[~hit].float() - y[~hit].float()).abs().max() <= 0.0625         # (fp32 sums in another order, one rounding: values up to 8)


@pytest.mark.parametrize("rows", [1, 2, 3, 4, 5, 6, 7, 8])
def test_runs_of_every_length_against_the_rotation(ss, rows):
    """One block of 16 images, six segments of `rows` rows, one workgroup each: rows + 6 input rows are 7 to 14 steps
    of a rotation of 7, from one whole turn with no rest to two."""
    N, H, W, C, k = 16, 6 * rows, 8, 640, 7
    rng = np.random.Generator(np.random.PCG64(rows))
    xb = wl.to_bits(rng.standard_normal((N, H, W, C), dtype=np.float32), wl.BF16)
    wb = wl.to_bits(rng.standard_normal((k, k, C), dtype=np.float32) * np.float32((2.0 / (k * k)) ** 0.5), wl.BF16)
    bias = (rng.standard_normal(C) * 0.1).astype(np.float32)
    y = _run(ss, xb, wb, bias, wl.BF16, (k // 2, k // 2), wl.ACT_RELU)
    check_close(y, oracle.dwconv2d(xb, wb, dtype=wl.BF16, bias=bias, pad=(k // 2, k // 2), act=wl.ACT_RELU), f"rows {rows}")


@pytest.mark.parametrize("H,W,C", [(1, 54_000_000, 8), (3, 1_400_000, 160)])
def test_few_rows_of_gigabytes(ss, H, W, C):
    """Padding rows and the image's own together pass 2 GiB: columns outside the image stay zero on either side (ones everywhere: each output counts
    the pixels of its window)."""
    x, w = torch.ones((1, H, W, C), dtype=torch.float16, device="cuda"), torch.ones((7, 7, C), dtype=torch.float16, device="cuda")
    assert x.numel() * 2 < 1 << 31 <= (H + 2) * W * C * 2
    y = ss.ss_dwconv2d_fwd(x, w, None, (3, 3), wl.ACT_NONE)
    for h in range(H):
        rows = min(h + 3, H - 1) - max(h - 3, 0) + 1
        want = rows * torch.tensor([4., 5., 6., 7., 7.], device="cuda")[:, None]
        assert torch.equal(y[0, h, :5].float(), want.expand(5, C)) and torch.equal(y[0, h, -5:].float(), want.flip(0).expand(5, C))
    assert bool((y[0, 0, 5:-5] == 7 * min(4, H)).all())
