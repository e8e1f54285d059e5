"""The workspace query on the host (it plans for 256 compute units where there is no device): a size where the library would split
a reduction over workgroups, none where the few-pixel kernels take the layer in both forms or the grid is large."""
import pytest

import paper_2411_00288_amd as ss


@pytest.mark.parametrize("dtype", [ss.SS_F16, ss.SS_BF16])
@pytest.mark.parametrize("N,splits", [(1, False), (2, False), (4, False), (8, False), (16, True), (24, True), (40, True), (64, False)])
def test_query_answers_for_the_kernel_that_runs(N, splits, dtype):
    desc = ss.make_desc(512, 512, 3, 3, dtype)
    need = ss.ss_conv2d_workspace_bytes(desc, N, 7, 7, (1, 1), (1, 1))
    assert (need > 0) == splits and need % 256 == 0


@pytest.mark.parametrize("N,image,cout,cin", [(83, 5, 256, 512), (24, 7, 512, 512), (40, 7, 512, 512), (3, 20, 256, 384)])
def test_layers_of_the_split_tests_split(N, image, cout, cin):
    assert ss.ss_conv2d_workspace_bytes(ss.make_desc(cout, cin, 3, 3, ss.SS_BF16), N, image, image, (1, 1), (1, 1)) > 0


def test_no_other_small_layer_asks_for_a_workspace():
    for cout, cin, k in [(64, 64, 3), (256, 256, 3), (2048, 512, 1), (512, 2048, 1), (512, 1024, 1), (136, 80, 3)]:
        for N in (1, 2, 4):
            assert ss.ss_conv2d_workspace_bytes(ss.make_desc(cout, cin, k, k, ss.SS_BF16), N, 14, 14, (1, 1), (k // 2,) * 2) == 0
