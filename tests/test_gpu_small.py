"""The kernels for few output pixels (tile ids 20 to 22): every staging mode, ragged tiles in both directions, reductions shorter and
longer than the waves' shares, all operand types, against the oracle; and the library's own choice of them under a HIP graph."""
import numpy as np
import pytest
import torch

import oracle
from paper_2411_00288_amd import workloads as wl
from helpers import check_close, dev_bits, layer_desc, oracle_ref, run_gpu

pytestmark = pytest.mark.gpu


def L_(N, H, W, cin, cout, k, s=1, p=0, dtype=wl.F16, korder=wl.K_CRS, act=wl.ACT_RELU, seed=21):
    return wl.Layer(f"n{N}h{H}w{W}c{cin}o{cout}k{k}s{s}d{dtype}o{korder}", N=N, H=H, W=W, cin=cin, cout=cout, kh=k, kw=k, stride=s,
                    pad=p, dtype=dtype, korder=korder, act=act, mask="logits", seed=seed)


SHAPES = [
    L_(1, 5, 7, 8, 20, 1), L_(1, 7, 7, 136, 40, 1, dtype=wl.BF16), L_(2, 6, 5, 520, 70, 1), L_(1, 3, 11, 2048, 33, 1, dtype=wl.BF16),
    L_(1, 9, 9, 64, 36, 1, s=2, p=1),
    L_(1, 6, 7, 24, 38, 3, p=1, korder=wl.K_RSC), L_(1, 9, 5, 104, 64, 3, s=2, p=1, korder=wl.K_RSC, dtype=wl.BF16),
    L_(1, 5, 5, 8, 16, 5, p=2, korder=wl.K_RSC),
    L_(1, 6, 7, 32, 40, 3, p=1), L_(2, 5, 5, 96, 66, 3, s=2, p=1, dtype=wl.BF16), L_(1, 7, 7, 288, 100, 3, p=1),
    L_(1, 5, 9, 76, 35, 3, p=1, dtype=wl.BF16), L_(1, 6, 6, 12, 64, 3, p=1),
    L_(1, 8, 6, 64, 40, 2, s=2), L_(1, 8, 10, 84, 36, 2, s=2, dtype=wl.BF16), L_(1, 4, 18, 352, 32, 2, s=2),
]


@pytest.mark.parametrize("sparse", [True, False])
@pytest.mark.parametrize("tile", [20, 21, 22])
@pytest.mark.parametrize("L", SHAPES, ids=lambda L: L.name)
def test_small_grid_kernels_match_oracle(ss, force_tile, L, tile, sparse):
    d = wl.make_inputs(L)
    force_tile(tile)
    check_close(run_gpu(ss, L, d, sparse=sparse), oracle_ref(L, d), L.name)


@pytest.mark.parametrize("act", [wl.ACT_RELU, wl.ACT_GELU])
@pytest.mark.parametrize("cout", [40, 38, 33])
@pytest.mark.parametrize("tile", [20, 22])
def test_small_grid_kernels_with_a_residual(ss, force_tile, tile, cout, act):
    L = L_(1, 6, 7, 64, cout, 3, p=1, dtype=wl.BF16, act=act)
    d = wl.make_inputs(L)
    res = wl.to_bits(np.random.Generator(np.random.PCG64(3)).standard_normal((1, L.Ho, L.Wo, cout), dtype=np.float32), L.dtype)
    desc = layer_desc(ss, L)
    packed = ss.ss_mask_compress(desc, dev_bits(d["W"], L.dtype), torch.from_numpy(d["M"]).cuda())
    force_tile(tile)
    y = ss.ss_conv2d_res_fwd(desc, dev_bits(d["x"], L.dtype), packed, torch.from_numpy(d["bias"]).cuda(), dev_bits(res, L.dtype), (1, 1),
                             (1, 1), act)
    check_close(y, oracle.conv2d(d["x"], d["W"], d["M"], cin=L.cin, kh=3, kw=3, korder=L.korder, dtype=L.dtype, bias=d["bias"],
                                 stride=(1, 1), pad=(1, 1), act=act, residual=res), L.name)


# Pointwise shares: exactly a ring of whole steps (256, 512: 2 and 4 waves), more than a ring from an odd step (2304 over 8 waves, 2560
# over 16: nine and five steps each), a share that ends early (480), a last step that is not whole (504, 2568).
@pytest.mark.parametrize("sparse", [True, False])
@pytest.mark.parametrize("tile", [20, 21, 22])
@pytest.mark.parametrize("cin,cout,s", [(256, 64, 1), (480, 38, 1), (504, 33, 1), (512, 68, 2), (2304, 36, 1), (2560, 40, 1), (2568, 34, 2)])
def test_pointwise_shares_of_whole_and_ragged_steps(ss, force_tile, cin, cout, s, tile, sparse):
    L = L_(1, 7, 9, cin, cout, 1, s=s, dtype=wl.BF16 if cin % 64 else wl.F16)
    d = wl.make_inputs(L)
    res = wl.to_bits(np.random.Generator(np.random.PCG64(5)).standard_normal((1, L.Ho, L.Wo, cout), dtype=np.float32), L.dtype)
    desc = layer_desc(ss, L)
    pack, run = (ss.ss_mask_compress, ss.ss_conv2d_res_fwd) if sparse else (ss.ss_dense_pack, ss.ss_conv2d_dense_res_fwd)
    w = pack(desc, dev_bits(d["W"], L.dtype), torch.from_numpy(d["M"]).cuda())
    force_tile(tile)
    y = run(desc, dev_bits(d["x"], L.dtype), w, torch.from_numpy(d["bias"]).cuda(), dev_bits(res, L.dtype), (s, s), (0, 0), L.act)
    check_close(y, oracle.conv2d(d["x"], d["W"], d["M"], cin=cin, kh=1, kw=1, korder=L.korder, dtype=L.dtype, bias=d["bias"],
                                 stride=(s, s), pad=(0, 0), act=L.act, residual=res), L.name)


@pytest.mark.parametrize("tile", [20, 21, 22])
@pytest.mark.parametrize("f8", [False, True])
@pytest.mark.parametrize("cin,k,korder", [(64, 3, wl.K_CRS), (320, 3, wl.K_CRS), (48, 3, wl.K_RSC), (1040, 1, wl.K_CRS), (192, 2, wl.K_CRS),
                                          (1024, 1, wl.K_CRS), (4608, 1, wl.K_CRS)])
def test_small_grid_kernels_on_8_bit_operands(ss, force_tile, cin, k, korder, f8, tile):
    L = L_(1, 6, 7, cin, 44, k, p=k // 2, dtype=wl.F8 if f8 else wl.I8, korder=korder)
    d = (wl.make_inputs_f8 if f8 else wl.make_inputs_q8)(L)
    desc = layer_desc(ss, L)
    t = {n: torch.from_numpy(d[n]).cuda() for n in ("W", "M", "x", "scale", "bias")}
    outs = []
    for tid in (2, tile):             # against a tiled kernel, itself checked against the oracle
        force_tile(tid)
        outs.append([ss.ss_conv2d_q8_fwd(desc, t["x"], ss.ss_mask_compress(desc, t["W"], t["M"]), t["scale"], t["bias"], (1, 1), (L.pad,) * 2, L.act),
                     ss.ss_conv2d_q8_dense_fwd(desc, t["x"], ss.ss_dense_pack(desc, t["W"], t["M"]), t["scale"], t["bias"], (1, 1), (L.pad,) * 2, L.act)])
    for a, b in zip(*outs):
        if f8:
            assert (torch.linalg.norm(a.float() - b.float()) / torch.linalg.norm(a.float())).item() <= 5e-4
        else:
            assert torch.equal(a, b)                          # integer sums are exact


def test_small_grid_choice_replays_in_a_hip_graph(ss):
    L = L_(1, 14, 14, 256, 256, 3, p=1, dtype=wl.BF16)
    d = wl.make_inputs(L)
    desc = layer_desc(ss, L)
    x = dev_bits(d["x"], L.dtype)
    packed = ss.ss_mask_compress(desc, dev_bits(d["W"], L.dtype), torch.from_numpy(d["M"]).cuda())
    launch, y = ss.prepare_conv2d(desc, x, packed, torch.from_numpy(d["bias"]).cuda(), (1, 1), (1, 1), L.act)
    launch()
    torch.cuda.synchronize()
    eager = y.clone()
    check_close(eager, oracle_ref(L, d), L.name)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        launch()
    for _ in range(3):
        y.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y.view(torch.int16), eager.view(torch.int16))


@pytest.mark.parametrize("tile", [20, 21, None])
@pytest.mark.parametrize("cin,mid,cout,s,H", [(32, 32, 32, 1, 5), (64, 64, 256, 1, 7), (96, 96, 160, 2, 9), (128, 128, 512, 1, 6), (32, 160, 64, 1, 5),
                                              (128, 256, 288, 2, 7)])
@pytest.mark.parametrize("sparse", [True, False])
def test_small_fused_pair_equals_the_two_calls(ss, force_tile, cin, mid, cout, s, H, sparse, tile):
    L1, L2 = L_(1, H, H + 2, cin, mid, 3, s=s, p=1, dtype=wl.BF16), L_(1, 1, 1, mid, cout, 1, dtype=wl.BF16, seed=22)
    a, b = wl.make_inputs(L1), wl.make_inputs(L2)
    d1, d2 = layer_desc(ss, L1), layer_desc(ss, L2)
    pack = (lambda d, t: ss.ss_mask_compress(d, dev_bits(t["W"], wl.BF16), torch.from_numpy(t["M"]).cuda())) if sparse else \
           (lambda d, t: ss.ss_dense_pack(d, dev_bits(t["W"], wl.BF16), torch.from_numpy(t["M"]).cuda()))
    w1, w2, b1, b2 = pack(d1, a), pack(d2, b), torch.from_numpy(a["bias"]).cuda(), torch.from_numpy(b["bias"]).cuda()
    x = dev_bits(a["x"], wl.BF16)
    res = torch.randn((1, L1.Ho, L1.Wo, cout), device="cuda").to(torch.bfloat16)
    force_tile(2)                                             # the two calls in tiled kernels
    conv, conv_res = (ss.ss_conv2d_fwd, ss.ss_conv2d_res_fwd) if sparse else (ss.ss_conv2d_dense_fwd, ss.ss_conv2d_dense_res_fwd)
    t = conv(d1, x, w1, b1, (s, s), (1, 1), wl.ACT_RELU)
    want = conv_res(d2, t, w2, b2, res, (1, 1), (0, 0), wl.ACT_GELU)
    force_tile(tile)
    fused = ss.ss_conv2d_pw_fused_fwd if sparse else ss.ss_conv2d_pw_fused_dense_fwd
    got = fused(d1, x, w1, b1, (s, s), (1, 1), wl.ACT_RELU, d2, w2, b2, res, wl.ACT_GELU)
    assert (torch.linalg.norm(got.float() - want.float()) / torch.linalg.norm(want.float())).item() <= 2e-3
