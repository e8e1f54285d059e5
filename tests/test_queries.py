"""What the library's queries answer, without a device: the sizes that the calls refuse, and where a joined call pays."""
import pytest

import paper_2411_00288_amd as ss
from paper_2411_00288_amd import workloads as wl


def _desc(cout, cin, k, korder=wl.K_CRS):
    return ss.make_desc(cout, cin, k, k, wl.BF16, korder)


def _joined(c1, c2, c3, image, sparse=True, N=1, cin=None):
    return ss.ss_conv2d_pw2_fused_query(_desc(c1, cin or c1, 3), (N, image, image), (1, 1), (1, 1), _desc(c2, c1, 1), _desc(c3, c2, 1), sparse)


@pytest.mark.parametrize("image", [7, 14, 28, 56])
def test_joined_layers_that_the_few_pixel_kernel_does_not_take_do_not_pay(image):
    for c1, c2, c3 in ((96, 384, 96), (64, 1024, 64), (128, 640, 128), (64, 256, 32), (128, 512, 32), (32, 256, 64), (32, 512, 128)):
        for sparse in (True, False):
            assert _joined(c1, c2, c3, image, sparse) == (True, False), (c1, c2, c3, sparse)
    for c1, c2, c3 in ((64, 256, 64), (64, 256, 128), (64, 512, 96), (128, 512, 128), (128, 512, 64)):
        assert _joined(c1, c2, c3, image) == (True, True)
        assert _joined(c1, c2, c3, image, False) == (True, c1 == 64)      # (the dense pair itself pays up to 64 channels)
    assert _joined(32, 128, 64, image) == (True, True) and _joined(32, 128, 64, image, False) == (True, False)
    # the third layer's rows need LDS too: with 16 pixels to a workgroup 352 input channels fit, with 32 128
    for N, limit in ((1, 352), (6272 // image ** 2, 128)):
        assert [_joined(128, 512, 128, image, N=N, cin=c) for c in (limit, limit + 32)] == [(True, True), (True, False)]


def test_joined_layers_on_more_pixels():
    # past one workgroup of 32 pixels per compute unit; past one of 64, where the pair of 128 channels loses its producer waves
    assert [_joined(96, 384, 96, 64, N=n)[1] for n in (2, 4, 5)] == [False, False, True]
    assert [_joined(128, 512, 128, 64, N=n)[1] for n in (2, 4, 5)] == [True, False, True]
    assert [_joined(64, 1024, 64, 64, N=n)[1] for n in (2, 3)] == [False, True]
    assert [_joined(64, 256, c3, 64, False, N=4)[1] for c3 in (64, 96)] == [True, False]


def test_pooled_layer_is_not_promised_where_the_call_refuses_it():
    q = lambda cout, N, H, W, pad=3: ss.ss_conv2d_maxpool_dense_query(_desc(cout, 4, 7, wl.K_RSC), (N, H, W), (2, 2), (pad, pad))
    # inputs of 2^31 - 2^26 bytes (992 images of 512 x 512) and more; padding rows of 2^26 bytes
    assert [q(8, n, 512, 512) for n in (991, 992, 1000)] == [True, False, False]
    assert [q(64, 1, 64, 512, p) for p in (3, 1500, 15000)] == [True, True, False]


def test_joined_layers_are_not_promised_where_the_call_refuses_them():
    # outputs of 2^31 elements, an input of 2^31 - 2^26 bytes
    assert [_joined(64, 256, 64, 2048, N=n)[0] for n in (1, 2)] == [True, False]
    assert [_joined(32, 128, 32, 1024, N=n, cin=512)[0] for n in (1, 2)] == [True, False]
