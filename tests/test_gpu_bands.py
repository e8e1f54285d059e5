"""Stores and loads end where the tensors end: operands and outputs that lie inside larger allocations, whose other elements keep their pattern (outputs)
or are NaN (inputs), at pixel counts that fill the last tile by any part."""
import numpy as np
import pytest
import torch

import oracle
from helpers import check_close, dev_bits, host_bits, layer_desc
from paper_2411_00288_amd import workloads as wl

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
