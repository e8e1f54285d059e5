"""A fused pair and the 1x1 layer behind it in one kernel (ss_conv2d_pw2_fused_fwd and its dense twin): the pair's output against the oracle's two
layers, the third layer's against the oracle applied to the output that the GPU stored; the tiled kernel (tile id 2 forced) and those for few
pixels (20, 21), widths that leave waves without rows or shares, pixel tails, strides; the trunk with and without it."""
import numpy as np
import pytest
import torch

import oracle
from helpers import check_close, dev_bits, host_bits
from paper_2411_00288_amd import workloads as wl
from test_gpu_fused import _oracle_pair, _pair

pytestmark = pytest.mark.gpu

# N, H, W, cin, first, second and third width, stride
SHAPES = [(1, 14, 14, 64, 64, 256, 64, 1), (2, 9, 11, 64, 128, 512, 128, 1), (1, 13, 5, 32, 32, 128, 32, 1), (1, 8, 8, 96, 64, 256, 128, 2),
          (3, 7, 7, 32, 96, 384, 96, 1), (1, 1, 1, 64, 64, 128, 96, 1), (1, 5, 13, 128, 128, 256, 64, 1)]


def _chain(ss, L1, L2, L3, d, res_bits, sparse):
    descs = [ss.make_desc(L.cout, L.cin, L.kh, L.kw, L.dtype, L.korder) for L in (L1, L2, L3)]
    pack = ss.ss_mask_compress if sparse else ss.ss_dense_pack
    w = [pack(dsc, dev_bits(e["W"], L1.dtype), torch.from_numpy(e["M"]).cuda()) for dsc, e in zip(descs, d)]
    b = [torch.from_numpy(e["bias"]).cuda() for e in d]
    res = None if res_bits is None else dev_bits(res_bits, L1.dtype)
    f = ss.ss_conv2d_pw2_fused_fwd if sparse else ss.ss_conv2d_pw2_fused_dense_fwd
    y2, y3 = f(descs[0], dev_bits(d[0]["x"], L1.dtype), w[0], b[0], (L1.stride,) * 2, (1, 1), L1.act, descs[1], w[1], b[1], res, L2.act, descs[2], w[2],
               None if L3.act == wl.ACT_NONE else b[2], L3.act)
    torch.cuda.synchronize()
    return y2, y3


@pytest.mark.parametrize("shape", SHAPES, ids=str)
@pytest.mark.parametrize("tile", [None, 2, 20, 21])
def test_against_oracle(ss, force_tile, tile, shape):
    N, H, W, cin, c1, c2, c3, s = shape
    i = SHAPES.index(shape)
    dtype = (wl.BF16, wl.F16)[i % 2]
    L1, L2 = _pair(N, H, W, cin, c1, c2, s=s, dtype=dtype, act2=(wl.ACT_RELU, wl.ACT_NONE)[i % 2], seed=70 + i)
    L3 = wl.Layer("third", N=N, H=L1.Ho, W=L1.Wo, cin=c2, cout=c3, kh=1, kw=1, dtype=dtype, act=(wl.ACT_RELU, wl.ACT_GELU, wl.ACT_NONE)[i % 3], mask="logits",
                  seed=170 + i)
    d = [wl.make_inputs(L) for L in (L1, L2, L3)]
    res = None if i == 4 else wl.to_bits(np.random.default_rng(i).standard_normal((N, L1.Ho, L1.Wo, c2)).astype(np.float32), dtype)
    _t, ref2 = _oracle_pair(L1, L2, d[0], d[1], res)
    force_tile(tile)
    for sparse in (True, False):
        y2, y3 = _chain(ss, L1, L2, L3, d, res, sparse)
        what = f"{shape} tile {tile} sparse {sparse}"
        got = y2.float().cpu().numpy().astype(np.float64)
        # (two layers' roundings, as in test_fused_pair_matches_oracle_chain)
        assert np.isfinite(got).all() and np.linalg.norm(got - ref2) <= 4e-3 * np.linalg.norm(ref2), what
        assert (np.abs(got - ref2) <= 2e-2 * (np.abs(ref2) + 1)).all(), what
        ref3 = oracle.conv2d(host_bits(y2), d[2]["W"], d[2]["M"], cin=c2, kh=1, kw=1, korder=L3.korder, dtype=dtype,
                             bias=None if L3.act == wl.ACT_NONE else d[2]["bias"], act=L3.act)
        check_close(y3, ref3, what + " (third layer on the GPU's own input)")


def test_refused_and_queried(ss):
    d = lambda cout, cin, k, korder=wl.K_CRS: ss.make_desc(cout, cin, k, k, wl.BF16, korder)
    q = lambda a, b, c, sparse=True, N=1: ss.ss_conv2d_pw2_fused_query(a, (N, 28, 28), (1, 1), (1, 1), b, c, sparse)
    w64, w128 = (d(64, 64, 3), d(256, 64, 1), d(64, 256, 1)), (d(128, 128, 3), d(512, 128, 1), d(128, 512, 1))
    assert q(*w64) == (True, True) and q(*w128) == (True, True) and q(*w128, False) == (True, False)
    assert [q(*w128, True, N)[1] for N in (10, 11, 20, 21)] == [True, False, False, True]      # few pixels; one 64-pixel workgroup per unit; more
    assert [q(*w64, sparse, 64)[1] for sparse in (True, False)] == [True, True] and q(d(64, 64, 3), d(256, 64, 1), d(128, 256, 1), False, 64) == (True, False)
    refused = [(d(128, 128, 3), d(512, 128, 1), d(256, 512, 1)), (d(64, 64, 3), d(224, 64, 1), d(64, 224, 1)), (d(64, 64, 3), d(256, 64, 1), d(48, 256, 1)),
               (d(64, 64, 3, wl.K_RSC), d(256, 64, 1), d(64, 256, 1)), (d(160, 64, 3), d(256, 160, 1), d(64, 256, 1)), (d(384, 96, 1), d(128, 384, 1), d(64, 128, 1))]
    for a, b, c in refused:
        stride_pad = ((1, 1), (a.kh // 2,) * 2)
        assert ss.ss_conv2d_pw2_fused_query(a, (1, 4, 4), *stride_pad, b, c, True) == (False, False)
        x = torch.zeros((1, 4, 4, a.cin), dtype=torch.bfloat16, device="cuda")
        w = [torch.zeros(ss.ss_packed_bytes(t), dtype=torch.uint8, device="cuda") for t in (a, b, c)]
        with pytest.raises(ss.SSError) as e:
            ss.ss_conv2d_pw2_fused_fwd(a, x, w[0], None, *stride_pad, 0, b, w[1], None, None, 0, c, w[2])
        assert e.value.status == ss.SS_ERR_UNSUPPORTED
    a, b, c = d(64, 64, 3), d(256, 64, 1), d(64, 128, 1)      # the third layer reads other channels
    with pytest.raises(ss.SSError) as e:
        q(a, b, c)
    assert e.value.status == ss.SS_ERR_INVALID_ARG


@pytest.mark.parametrize("batch,image,sparse,joined_layers", [(1, 64, True, 6), (1, 64, False, 3), (5, 224, True, 6), (5, 224, False, 2)])
def test_trunk_with_joined_layers_equals_its_single_launches(ss, batch, image, sparse, joined_layers):
    """Every buffer that the joined kernels write, against the pair's and the layer's own launches."""
    from paper_2411_00288_amd import resnet50
    t = resnet50.Trunk(batch=batch, image=image, dtype=wl.BF16, sparse=sparse)
    assert len(t.launches) - len(t.chain) == joined_layers + 1      # (and the pooling)
    t.input.copy_(torch.randn(t.input.shape, device="cuda").to(torch.bfloat16))
    t.forward()
    torch.cuda.synchronize()
    joined = {i: b.clone() for i, b in t.bufs.items()}
    for b in list(t.bufs.values())[1:]:
        b.fill_(float("nan"))
    for launch in t.launches:
        launch()
    torch.cuda.synchronize()
    single = {op.dst for op in t.ops if op.name in t.fused}
    for op in t.ops:
        if op.dst in single:
            continue                                      # (a fused pair's 3x3: never written)
        a, b = joined[op.dst].float(), t.bufs[op.dst].float()
        assert torch.isfinite(a).all() and (torch.linalg.norm(a - b) <= 1e-2 * torch.linalg.norm(b)).item(), op.name
