"""A fused pair and the 1x1 layer behind it in one kernel give the bits of the separate calls: the third layer's sums are formed in the shares and the
order of its own call, whichever kernel that call takes for the size (waves that share a reduction, one chain of products), the biases behind them."""
import pytest
import torch

from paper_2411_00288_amd import workloads as wl

pytestmark = pytest.mark.gpu

# first, second and third width
WIDTHS = [(64, 256, 64), (64, 256, 128), (128, 512, 128), (128, 512, 96), (64, 384, 96), (128, 384, 64), (64, 128, 64), (128, 512, 64)]


# pixels: workgroups of 16 and of 32, third layers of 128 and of 96 channels past the few-pixel kernels (one chain of products, of 16 steps over two
# waves), the last size with workgroups of 32, and the tiled kernel
@pytest.mark.parametrize("P", [37, 3136, 4500, 7001, 8192, 8193, 20001])
@pytest.mark.parametrize("sparse", [True, False])
def test_bits_of_the_separate_calls(ss, P, sparse):
    gen = torch.Generator(device="cuda").manual_seed(P)
    for i, (c1, c2, c3) in enumerate(WIDTHS):
        dtype = (wl.BF16, wl.F16)[i % 2]
        tdt = ss.torch_dtype(dtype)
        rand = lambda *shape: torch.randn(shape, device="cuda", generator=gen)
        layers = []
        for cout, cin, k in ((c1, 64, 3), (c2, c1, 1), (c3, c2, 1)):
            K = cin * k * k
            desc = ss.make_desc(cout, cin, k, k, dtype, wl.K_CRS)
            W = (rand(cout, K) * (2.0 / K) ** 0.5).to(tdt)
            M = torch.tensor([[1, 0, 0, 1], [0, 1, 1, 0]], dtype=torch.uint8, device="cuda").repeat((cout + 1) // 2, K // 4)[:cout].contiguous()
            layers.append((desc, ss.ss_mask_compress(desc, W, M) if sparse else ss.ss_dense_pack(desc, W, M), rand(cout) * 0.1))
        (d1, w1, b1), (d2, w2, b2), (d3, w3, b3) = layers
        x, res = rand(1, 1, P, 64).to(tdt), rand(1, 1, P, c2).to(tdt)
        act3 = (wl.ACT_RELU, wl.ACT_NONE, wl.ACT_GELU)[i % 3]
        pair, joined, conv = ((ss.ss_conv2d_pw_fused_fwd, ss.ss_conv2d_pw2_fused_fwd, ss.ss_conv2d_fwd) if sparse else
                              (ss.ss_conv2d_pw_fused_dense_fwd, ss.ss_conv2d_pw2_fused_dense_fwd, ss.ss_conv2d_dense_fwd))
        y2 = pair(d1, x, w1, b1, (1, 1), (1, 1), wl.ACT_RELU, d2, w2, b2, res, wl.ACT_RELU)
        y3 = conv(d3, y2, w3, b3, act=act3)
        j2, j3 = joined(d1, x, w1, b1, (1, 1), (1, 1), wl.ACT_RELU, d2, w2, b2, res, wl.ACT_RELU, d3, w3, b3, act3)
        what = (P, c1, c2, c3, sparse)
        assert torch.isfinite(y3).all() and torch.equal(j2.view(torch.int16), y2.view(torch.int16)), what
        assert torch.equal(j3.view(torch.int16), y3.view(torch.int16)), what


@pytest.mark.parametrize("batch,image,sparse", [(1, 64, True), (1, 224, True), (1, 224, False), (2, 224, True), (7, 224, True), (7, 224, False), (22, 224, True)])
def test_trunk_gives_the_bits_of_its_single_launches(ss, batch, image, sparse):
    from paper_2411_00288_amd import resnet50
    t = resnet50.Trunk(batch=batch, image=image, dtype=wl.BF16, sparse=sparse)
    t.input.copy_(torch.randn(t.input.shape, device="cuda").to(torch.bfloat16))
    t.forward()
    joined = {i: b.clone() for i, b in t.bufs.items()}
    for launch in t.launches:
        launch()
    differ = [op.name for op in t.ops if not torch.equal(joined[op.dst].view(torch.int16), t.bufs[op.dst].view(torch.int16))]
    assert differ == []
