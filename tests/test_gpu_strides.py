"""Strides that differ between the two directions (the other tests step alike in both), through every kernel that turns a pixel's number into a
place in the input, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from helpers import check_close, dev_bits, layer_desc
from paper_2411_00288_amd import workloads as wl

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
