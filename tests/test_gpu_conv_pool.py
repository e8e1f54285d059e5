"""The dense first layer of an image network and its 3x3 max pooling in one kernel (ss_conv2d_maxpool_dense_fwd): the layer's output against the
oracle, and bit for bit against its own call; the pooled output bit for bit against the pooling of what the GPU stored.  Sizes around the tile of 14 x 14
outputs (7 x 7 pooled), odd and even, output channels that fill no group of 64, NaN and infinities in the image."""
import numpy as np
import pytest
import torch

import oracle
from helpers import check_close, dev_bits, host_bits
from paper_2411_00288_amd import workloads as wl

pytestmark = pytest.mark.gpu

# N, H, W, channels, output channels
SHAPES = [(1, 1, 1, 4, 64), (1, 28, 28, 4, 64), (1, 29, 27, 3, 64), (1, 30, 31, 4, 64), (2, 57, 26, 3, 72), (1, 58, 59, 4, 8), (3, 13, 97, 3, 128)]


def _layer(shape, dtype, korder=wl.K_CRS):
    N, H, W, cin, cout = shape
    return wl.Layer("first", N=N, H=H, W=W, cin=cin, cout=cout, kh=7, kw=7, stride=2, pad=3, dtype=dtype, act=wl.ACT_RELU, korder=korder, mask="none",
                    relu_input=False, seed=sum(shape))


@pytest.mark.parametrize("special", [False, True])
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_against_oracle_and_the_two_calls(ss, shape, special):
    i = SHAPES.index(shape)
    dtype = (wl.BF16, wl.F16)[i % 2]
    L = _layer(shape, dtype, wl.K_RSC if shape[3] == 4 and i % 3 else wl.K_CRS)
    d = wl.make_inputs(L)
    if special:
        flat = d["x"].reshape(-1)
        pos = np.random.default_rng(i).integers(0, flat.size, 4)
        flat[pos] = wl.to_bits(np.array([np.inf, -np.inf, np.nan, 0], np.float32), dtype)
    desc = ss.make_desc(L.cout, L.cin, 7, 7, dtype, L.korder)
    w = ss.ss_dense_pack(desc, dev_bits(d["W"], dtype), None)
    x, bias = dev_bits(d["x"], dtype), torch.from_numpy(d["bias"]).cuda()
    assert ss.ss_conv2d_maxpool_dense_query(desc, (L.N, L.H, L.W), (2, 2), (3, 3))
    alone = ss.ss_conv2d_dense_fwd(desc, x, w, bias, (2, 2), (3, 3), L.act)
    y, pooled = torch.full_like(alone, float("nan")), torch.full_like(ss.ss_maxpool2d(alone, 3, 2, 1), float("nan"))
    for limit in (0, 1):                                       # many workgroups; two, each with many tiles
        ss.ss_debug_limit_blocks(limit)
        try:
            ss.ss_conv2d_maxpool_dense_fwd(desc, x, w, bias, (2, 2), (3, 3), y=y, pooled=pooled)
            torch.cuda.synchronize()
        finally:
            ss.ss_debug_limit_blocks(0)
        assert torch.equal(y.view(torch.int16), alone.view(torch.int16))
        assert torch.equal(pooled.view(torch.int16), ss.ss_maxpool2d(y, 3, 2, 1).view(torch.int16))
    if not special:
        check_close(y, oracle.conv2d(d["x"], d["W"], None, cin=L.cin, kh=7, kw=7, korder=L.korder, dtype=dtype, bias=d["bias"], stride=(2, 2), pad=(3, 3),
                                     act=L.act), str(shape))
        assert np.array_equal(host_bits(pooled), oracle.maxpool2d(host_bits(y), dtype=dtype, k=3, stride=2, pad=1))


def test_refused(ss):
    d = lambda **k: ss.make_desc(k.get("cout", 64), k.get("cin", 4), k.get("k", 7), k.get("k", 7), k.get("dtype", wl.BF16), wl.K_RSC)
    cases = [(d(), (1, 1), 3, ss.SS_ACT_RELU), (d(), (2, 2), 3, ss.SS_ACT_NONE), (d(), (2, 2), 3, ss.SS_ACT_GELU), (d(k=5), (2, 2), 2, ss.SS_ACT_RELU),
             (d(cin=8), (2, 2), 3, ss.SS_ACT_RELU), (d(cout=60), (2, 2), 3, ss.SS_ACT_RELU)]
    for desc, stride, pad, act in cases:
        assert not ss.ss_conv2d_maxpool_dense_query(desc, (1, 16, 16), stride, (pad,) * 2, act)
        x = torch.zeros((1, 16, 16, desc.cin), dtype=torch.bfloat16, device="cuda")
        w = torch.zeros(ss.ss_dense_bytes(desc), dtype=torch.uint8, device="cuda")
        with pytest.raises(ss.SSError) as e:
            ss.ss_conv2d_maxpool_dense_fwd(desc, x, w, None, stride, (pad,) * 2, act)
        assert e.value.status == ss.SS_ERR_UNSUPPORTED
    # y of 2^31 - 2^27 bytes and one image less
    assert [ss.ss_conv2d_maxpool_dense_query(d(), (n, 256, 256), (2, 2), (3, 3)) for n in (960, 959)] == [False, True]
    with pytest.raises(ss.SSError) as e:
        ss.ss_conv2d_maxpool_dense_query(d(), (1, 0, 4), (2, 2), (3, 3))
    assert e.value.status == ss.SS_ERR_INVALID_ARG
