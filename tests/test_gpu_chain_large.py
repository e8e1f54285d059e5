"""The joined pair and third layer on residuals either side of the line from which they are read with the non-temporal hint (72 MiB): the launch
on all images against launches on single ones, bit for bit (a pixel's sums do not depend on its tile)."""
import pytest
import torch

from paper_2411_00288_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("images", [23, 24])
def test_all_images_equal_single_ones(ss, force_tile, images):
    H, dtype = 80, wl.BF16                                   # 6400 pixels, a whole number of tiles; 3.1 MiB of residual an image
    gen = torch.Generator(device="cuda").manual_seed(images)
    rand = lambda *shape: torch.randn(shape, device="cuda", generator=gen).to(torch.bfloat16) * 0.1
    layers = []
    for cout, cin, k in ((64, 64, 3), (256, 64, 1), (32, 256, 1)):
        desc = ss.make_desc(cout, cin, k, k, dtype, wl.K_CRS)
        layers.append((desc, ss.ss_dense_pack(desc, rand(cout, cin * k * k), None), torch.randn(cout, device="cuda", generator=gen)))
    x, res = rand(images, H, H, 64), rand(images, H, H, 256)
    assert (res.numel() * 2 >= 72 << 20) == (images == 24)
    force_tile(2)

    def run(x, res):
        (d1, w1, b1), (d2, w2, b2), (d3, w3, b3) = layers
        return ss.ss_conv2d_pw2_fused_dense_fwd(d1, x, w1, b1, (1, 1), (1, 1), wl.ACT_RELU, d2, w2, b2, res, wl.ACT_RELU, d3, w3, b3, wl.ACT_RELU)
    y2, y3 = run(x, res)
    for i in (0, images // 2, images - 1):
        one2, one3 = run(x[i:i + 1].contiguous(), res[i:i + 1].contiguous())
        assert torch.equal(y2[i:i + 1], one2) and torch.equal(y3[i:i + 1], one3)
    assert torch.isfinite(y3).all()
