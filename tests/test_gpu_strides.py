"""Strides that differ between the two directions (the other tests step alike in both), through every kernel that turns a pixel's number into a
place in the input, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from helpers import check_close, dev_bits, host_bits, layer_desc
from paper_2411_00288_amd import workloads as wl
from test_gpu_q8 import check_q8

pytestmark = pytest.mark.gpu


def _L(N, H, W, cin, cout, k=1, p=0, dtype=wl.F16, korder=wl.K_CRS, act=wl.ACT_RELU, seed=41):
    return wl.Layer(f"strides_n{N}h{H}w{W}c{cin}o{cout}k{k}p{p}d{dtype}o{korder}", N=N, H=H, W=W, cin=cin, cout=cout, kh=k, kw=k, pad=p,
                    dtype=dtype, korder=korder, act=act, mask="logits", seed=seed)


def _out(L, stride):
    return (L.H + 2 * L.pad - L.kh) // stride[0] + 1, (L.W + 2 * L.pad - L.kw) // stride[1] + 1


def _check(ss, L, stride, residual=False):
    d, desc = wl.make_inputs(L), layer_desc(ss, L)
    W, M, x, bias = dev_bits(d["W"], L.dtype), torch.from_numpy(d["M"]).cuda(), dev_bits(d["x"], L.dtype), torch.from_numpy(d["bias"]).cuda()
    res = None
    if residual:
        res = wl.to_bits(np.random.Generator(np.random.PCG64(3)).standard_normal((L.N, *_out(L, stride), L.cout), dtype=np.float32), L.dtype)
    ref = oracle.conv2d(d["x"], d["W"], d["M"], cin=L.cin, kh=L.kh, kw=L.kw, korder=L.korder, dtype=L.dtype, bias=d["bias"], stride=stride,
                        pad=(L.pad,) * 2, act=L.act, residual=res)
    for sparse in (True, False):
        w = ss.ss_mask_compress(desc, W, M) if sparse else ss.ss_dense_pack(desc, W, M)
        if res is None:
            y = (ss.ss_conv2d_fwd if sparse else ss.ss_conv2d_dense_fwd)(desc, x, w, bias, stride, (L.pad,) * 2, L.act)
        else:
            y = (ss.ss_conv2d_res_fwd if sparse else ss.ss_conv2d_dense_res_fwd)(desc, x, w, bias, dev_bits(res, L.dtype), stride, (L.pad,) * 2, L.act)
        check_close(y, ref, f"{L.name} stride {stride} sparse {sparse} residual {residual}")


@pytest.mark.parametrize("residual", [False, True])
@pytest.mark.parametrize("stride", [(1, 3), (3, 1), (3, 5), (1, 2), (2, 1)])
def test_activation_stationary_kernel(ss, force_tile, stride, residual):
    force_tile(13)
    _check(ss, _L(2, 13, 17, 64, 264, dtype=wl.BF16), stride, residual)
    _check(ss, _L(1, 16, 30, 256, 512), stride, residual)


@pytest.mark.parametrize("stride,H,W", [((1, 3), 64, 96), ((3, 1), 144, 32), ((3, 5), 150, 250)])
def test_choice_for_expanding_pointwise_layers(ss, stride, H, W):
    """Grids above the few-pixel kernels' range: the library takes the activation-stationary kernel by itself."""
    _check(ss, _L(2, H, W, 64, 256), stride)


@pytest.mark.parametrize("tile", [None, 20, 21, 22])
@pytest.mark.parametrize("stride", [(1, 3), (3, 1), (3, 5), (1, 2)])
def test_few_pixel_pointwise_kernels(ss, force_tile, stride, tile):
    force_tile(tile)
    _check(ss, _L(1, 9, 16, 128, 72), stride)
    _check(ss, _L(2, 7, 11, 72, 40, dtype=wl.BF16), stride, residual=True)


@pytest.mark.parametrize("tile", [None, 20, 21, 22])
@pytest.mark.parametrize("stride", [(1, 3), (3, 1), (3, 5), (1, 2)])
def test_few_pixel_pointwise_kernels_on_8_bit_operands(ss, force_tile, stride, tile):
    force_tile(tile)
    q, f = _L(1, 9, 16, 256, 72, dtype=wl.I8), _L(2, 7, 11, 128, 40, dtype=wl.F8)
    for L, d, reference, check in ((q, wl.make_inputs_q8(q), oracle.conv2d_q8, check_q8), (f, wl.make_inputs_f8(f), oracle.conv2d_f8, check_close)):
        desc = ss.make_desc(L.cout, L.cin, 1, 1, L.dtype, L.korder)
        x, W, M, scale, bias = (torch.from_numpy(d[k]).cuda() for k in ("x", "W", "M", "scale", "bias"))
        ref = reference(d["x"], d["W"], d["M"], cin=L.cin, kh=1, kw=1, korder=L.korder, scale=d["scale"], bias=d["bias"], stride=stride, act=L.act)
        check(ss.ss_conv2d_q8_fwd(desc, x, ss.ss_mask_compress(desc, W, M), scale, bias, stride, (0, 0), L.act), ref, f"{L.name} sparse")
        check(ss.ss_conv2d_q8_dense_fwd(desc, x, ss.ss_dense_pack(desc, W, M), scale, bias, stride, (0, 0), L.act), ref, f"{L.name} dense")


@pytest.mark.parametrize("stride", [(1, 2), (2, 3), (3, 1)])
@pytest.mark.parametrize("tile", [2, 4, 7, 10, 11])
def test_three_by_three(ss, force_tile, tile, stride):
    """Tiled, producer-wave and resident-grid kernels."""
    force_tile(tile)
    _check(ss, _L(2, 13, 15, 64, 264, k=3, p=1), stride)
    _check(ss, _L(1, 11, 14, 32, 136, k=2, dtype=wl.BF16), stride)
    if tile < 10:
        _check(ss, _L(1, 9, 16, 72, 130, k=3, p=1, korder=wl.K_RSC), stride, residual=True)
        _check(ss, _L(2, 9, 16, 192, 100, dtype=wl.BF16), stride)


@pytest.mark.parametrize("stride", [(1, 2), (2, 3), (3, 1)])
@pytest.mark.parametrize("tile", [2, 4, 20, 21])
def test_fused_pair(ss, force_tile, tile, stride):
    force_tile(tile)
    L1 = _L(2, 13, 15, 64, 128, k=3, p=1, dtype=wl.BF16)
    Ho, Wo = _out(L1, stride)
    L2 = _L(2, Ho, Wo, 128, 160, dtype=wl.BF16, act=wl.ACT_NONE, seed=43)
    d1, d2 = wl.make_inputs(L1), wl.make_inputs(L2)
    s1, s2 = layer_desc(ss, L1), layer_desc(ss, L2)
    x, b1, b2 = dev_bits(d1["x"], wl.BF16), torch.from_numpy(d1["bias"]).cuda(), torch.from_numpy(d2["bias"]).cuda()
    w1 = ss.ss_mask_compress(s1, dev_bits(d1["W"], wl.BF16), torch.from_numpy(d1["M"]).cuda())
    w2 = ss.ss_mask_compress(s2, dev_bits(d2["W"], wl.BF16), torch.from_numpy(d2["M"]).cuda())
    y = ss.ss_conv2d_pw_fused_fwd(s1, x, w1, b1, stride, (1, 1), L1.act, s2, w2, b2, None, L2.act)
    force_tile(0)
    t = ss.ss_conv2d_fwd(s1, x, w1, b1, stride, (1, 1), L1.act)
    check_close(t, oracle.conv2d(d1["x"], d1["W"], d1["M"], cin=64, kh=3, kw=3, korder=L1.korder, dtype=wl.BF16, bias=d1["bias"], stride=stride,
                                 pad=(1, 1), act=L1.act), "first layer")
    check_close(y, oracle.conv2d(host_bits(t), d2["W"], d2["M"], cin=128, kh=1, kw=1, korder=L2.korder, dtype=wl.BF16, bias=d2["bias"], act=L2.act),
                "second layer on the first one's output")
