"""Stores and loads end where the tensors end: operands and outputs that lie inside larger allocations, whose other elements keep their pattern (outputs)
or are NaN (inputs), at pixel counts that fill the last tile by any part."""
import numpy as np
import pytest
import torch

import oracle
from helpers import check_close, dev_bits, host_bits, layer_desc
from paper_2411_00288_amd import workloads as wl
from test_gpu_q8 import check_q8

pytestmark = pytest.mark.gpu

BAND = 1 << 16                                            # elements on either side: more than a tile of 128 pixels x 512 channels
PATTERN = 0x7FC3                                          # (a NaN in both 16-bit types)


class Banded:
    """A 16-bit tensor in the middle of an allocation whose other elements hold PATTERN."""

    def __init__(self, shape, dtype, bits=None):
        n = int(np.prod(shape))
        self.all = torch.full((n + 2 * BAND,), PATTERN, dtype=torch.int16, device="cuda")
        self.inner = self.all[BAND:BAND + n].view(shape).view(torch.float16 if dtype == wl.F16 else torch.bfloat16)
        if bits is not None:
            self.inner.view(torch.int16).copy_(torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)))

    def bands_are_whole(self):
        return bool((self.all[:BAND] == PATTERN).all() and (self.all[-BAND:] == PATTERN).all())


def _layer(P, cin, cout, k, dtype, act, seed):
    return wl.Layer(f"p{P}c{cin}o{cout}k{k}", N=1, H=1, W=P, cin=cin, cout=cout, kh=k, kw=k, pad=k // 2, dtype=dtype, act=act, mask="logits", seed=seed)


@pytest.mark.parametrize("residual", [False, True])
@pytest.mark.parametrize("P", [1, 15, 17, 64 + 31, 33, 63, 128])
def test_inverted_bottleneck(ss, P, residual):
    dtype = wl.BF16
    L1, L2 = _layer(P, 96, 384, 1, dtype, wl.ACT_GELU, P), _layer(P, 384, 96, 1, dtype, wl.ACT_NONE, P + 1)
    d1, d2 = wl.make_inputs(L1), wl.make_inputs(L2)
    s1, s2 = layer_desc(ss, L1), layer_desc(ss, L2)
    res = wl.to_bits(np.random.Generator(np.random.PCG64(2)).standard_normal((1, 1, P, 96), dtype=np.float32), dtype) if residual else None
    x, r, y = Banded((1, 1, P, 96), dtype, d1["x"]), Banded((1, 1, P, 96), dtype, res) if residual else None, Banded((1, 1, P, 96), dtype)
    W, M = [dev_bits(d["W"], dtype) for d in (d1, d2)], [torch.from_numpy(d["M"]).cuda() for d in (d1, d2)]
    b = [torch.from_numpy(d["bias"]).cuda() for d in (d1, d2)]
    for sparse in (True, False):
        pack = ss.ss_mask_compress if sparse else ss.ss_dense_pack
        w = [pack(s, W[i], M[i]) for i, s in enumerate((s1, s2))]
        t = (ss.ss_conv2d_fwd if sparse else ss.ss_conv2d_dense_fwd)(s1, x.inner, w[0], b[0], (1, 1), (0, 0), L1.act)
        (ss.ss_conv2d_pw_fused_fwd if sparse else ss.ss_conv2d_pw_fused_dense_fwd)(s1, x.inner, w[0], b[0], (1, 1), (0, 0), L1.act, s2, w[1], b[1],
                                                                                    r.inner if residual else None, L2.act, y.inner)
        assert y.bands_are_whole()
        check_close(y.inner, oracle.conv2d(host_bits(t), d2["W"], d2["M"], cin=384, kh=1, kw=1, korder=L2.korder, dtype=dtype, bias=d2["bias"],
                                           act=L2.act, residual=res), f"{P} pixels sparse {sparse}")


@pytest.mark.parametrize("k", [2, 3])
@pytest.mark.parametrize("tile", [10, 11])
@pytest.mark.parametrize("P", [1, 31, 33, 64 + 32, 127, 128 + 15])
def test_resident_grid_kernels(ss, force_tile, P, tile, k):
    dtype = wl.F16
    L = wl.Layer(f"p{P}k{k}t{tile}", N=1, H=k, W=P + k - 1, cin=64, cout=264, kh=k, kw=k, dtype=dtype, act=wl.ACT_RELU, mask="logits", seed=P)
    d, desc = wl.make_inputs(L), layer_desc(ss, L)
    x, y = Banded(d["x"].shape, dtype, d["x"]), Banded((1, 1, P, 264), dtype)
    W, M, b = dev_bits(d["W"], dtype), torch.from_numpy(d["M"]).cuda(), torch.from_numpy(d["bias"]).cuda()
    ref = oracle.conv2d(d["x"], d["W"], d["M"], cin=64, kh=k, kw=k, korder=L.korder, dtype=dtype, bias=d["bias"], act=L.act)
    force_tile(tile)
    for sparse in (True, False):
        w = (ss.ss_mask_compress if sparse else ss.ss_dense_pack)(desc, W, M)
        (ss.ss_conv2d_fwd if sparse else ss.ss_conv2d_dense_fwd)(desc, x.inner, w, b, (1, 1), (0, 0), L.act, y.inner)
        assert y.bands_are_whole()
        check_close(y.inner, ref, f"{P} pixels sparse {sparse}")


@pytest.mark.parametrize("dtype", [wl.I8, wl.F8])
@pytest.mark.parametrize("tile", [10, 11])
@pytest.mark.parametrize("P", [1, 31, 33, 64 + 32, 127, 128 + 15])
def test_resident_grid_kernels_on_8_bit_operands(ss, force_tile, P, tile, dtype):
    L = wl.Layer(f"p{P}t{tile}d{dtype}", N=1, H=3, W=P + 2, cin=64, cout=264, kh=3, kw=3, dtype=dtype, act=wl.ACT_RELU, mask="logits", seed=P)
    d = (wl.make_inputs_q8 if dtype == wl.I8 else wl.make_inputs_f8)(L)
    desc, y = ss.make_desc(264, 64, 3, 3, dtype, L.korder), Banded((1, 1, P, 264), wl.F16)
    x, W, M, scale, bias = (torch.from_numpy(d[k]).cuda() for k in ("x", "W", "M", "scale", "bias"))
    force_tile(tile)
    ss.ss_conv2d_q8_fwd(desc, x, ss.ss_mask_compress(desc, W, M), scale, bias, (1, 1), (0, 0), L.act, y.inner)
    assert y.bands_are_whole()
    reference, check = (oracle.conv2d_q8, check_q8) if dtype == wl.I8 else (oracle.conv2d_f8, check_close)
    check(y.inner, reference(d["x"], d["W"], d["M"], cin=64, kh=3, kw=3, korder=L.korder, scale=d["scale"], bias=d["bias"], act=L.act), L.name)


@pytest.mark.parametrize("P", [2049, 2049 + 31, 2049 + 62])
def test_activation_stationary_kernel(ss, force_tile, P):
    """(Its offsets were in the vector part already.)"""
    L = _layer(P, 64, 256, 1, wl.BF16, wl.ACT_RELU, P)
    d, desc = wl.make_inputs(L), layer_desc(ss, L)
    res = wl.to_bits(np.random.Generator(np.random.PCG64(2)).standard_normal((1, 1, P, 256), dtype=np.float32), L.dtype)
    x, r, y = Banded((1, 1, P, 64), L.dtype, d["x"]), Banded((1, 1, P, 256), L.dtype, res), Banded((1, 1, P, 256), L.dtype)
    w = ss.ss_mask_compress(desc, dev_bits(d["W"], L.dtype), torch.from_numpy(d["M"]).cuda())
    force_tile(13)
    ss.ss_conv2d_res_fwd(desc, x.inner, w, torch.from_numpy(d["bias"]).cuda(), r.inner, (1, 1), (0, 0), L.act, y.inner)
    assert y.bands_are_whole()
    check_close(y.inner, oracle.conv2d(d["x"], d["W"], d["M"], cin=64, kh=1, kw=1, korder=L.korder, dtype=L.dtype, bias=d["bias"], act=L.act,
                                       residual=res), L.name)
