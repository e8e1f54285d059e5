"""The tile of channels-last layers with short reductions (choose_vec_short), on the host and on the GPU against the 128-row tile."""
import shutil
import subprocess
from pathlib import Path

import pytest
import torch

import test_gpu_f8 as f8
import test_gpu_q8 as q8
import test_gpu_tail as tail
from helpers import run_gpu
from paper_2411_00288_amd import workloads as wl

ROOT = Path(__file__).resolve().parent.parent
LARGE = 64 * 256 * 40


def test_both_sides_of_the_lines(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    exe = tmp_path / "choose_vec_short"
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", str(ROOT / "include"),
                    str(ROOT / "tests" / "host" / "choose_vec_short.cpp"), "-o", str(exe)], check=True, capture_output=True)
    # (channels, pixels, bytes, sparse, f8)
    want = {}
    for kind in ((0, 1, 0), (1, 1, 0), (1, 1, 1)):
        want.update({(c, LARGE) + kind: t for c, t in ((96, 2), (128, 2), (129, 7), (160, 7), (161, 2), (288, 2))})
    for kind in ((0, 0, 0), (1, 0, 0)):
        want.update({(c, LARGE) + kind: t for c, t in ((65, 6), (96, 6), (97, 2), (128, 2), (129, 6), (192, 6), (193, 2), (256, 2), (257, 6), (288, 6), (289, 2), (448, 2))})
    want.update({(c, LARGE, 1, 0, 1): 2 for c in (96, 160, 288)})
    # 96 rows by workgroups per compute unit (one tile of rows)
    for kind, lo in (((0, 0, 0), 3), ((1, 0, 0), 2), ((0, 1, 0), 3), ((1, 1, 1), 3)):
        sparse = kind[1]
        want.update({(96, 64 * 256 * n + more) + kind: t for n, more, t in ((lo, 0, 2), (lo, 1, 6), (5, 0, 6), (5, 1, 2), (6, 0, 2), (6, 1, 2 if sparse else 6))})
    want.update({(64, LARGE, 1, 0, 0): 0, (136, 64 * 129, 0, 1, 0): 5, (136, 64 * 128, 0, 1, 0): 4})      # the others keep theirs
    out = subprocess.run([str(exe)], input="".join("%d %d %d %d %d\n" % k for k in want), capture_output=True, text=True, check=True).stdout.split()
    assert [int(o) for o in out] == list(want.values())


# (channels, height, width, tile of the sparse and of the dense layers): a last tile of one pixel, 401, 307, 801 and 1538 tiles of pixels, where the library takes
# other tiles than the 128 rows they are compared with (not for dense FP8); K below 512 in 2-byte units and no multiple of a step
@pytest.mark.gpu
@pytest.mark.parametrize("cout,H,W,sparse_tile,dense_tile", [(129, 1, 25601, 7, 6), (160, 1, 25601, 7, 6), (192, 1, 25601, 6, 6), (257, 1, 19585, 6, 6),
                                                             (280, 1, 19585, 6, 6), (66, 3, 17067, 6, 6), (96, 3, 17067, 6, 6), (96, 1, 98369, 2, 6)])
def test_choice_against_128_rows(ss, force_tile, cout, H, W, sparse_tile, dense_tile):
    for sparse in (True, False):
        if (sparse_tile if sparse else dense_tile) == 2:
            continue                                      # (the same kernel twice)
        for mod, make, cin in ((q8, wl.make_inputs_q8, 48), (f8, wl.make_inputs_f8, 48), (None, wl.make_inputs, 24)):
            if mod is f8 and not sparse:
                continue
            L = (mod or tail)._L(1, H, W, cin, cout, 3, p=1, korder=wl.K_RSC, seed=cout, **({} if mod else {"dtype": wl.BF16, "act": wl.ACT_RELU}))
            d = make(L)
            out = []
            for tile in (None, sparse_tile if sparse else dense_tile, 2):
                force_tile(tile)
                out.append(mod._run(ss, L, d, sparse=sparse) if mod else run_gpu(ss, L, d, sparse=sparse))
            y, named, ref = (o if isinstance(o, torch.Tensor) else torch.as_tensor(o) for o in out)
            # every height adds a row's products in the same order and has the same epilogue
            for o in (named, ref):
                assert torch.equal(y.contiguous().view(torch.uint8), o.contiguous().view(torch.uint8)), f"{L.name} sparse {sparse}"


@pytest.mark.gpu
@pytest.mark.parametrize("cout,H,W", [(129, 1, 25601), (160, 1, 25601), (280, 1, 19585), (96, 3, 17067)])
def test_choice_against_128_rows_with_a_residual(ss, force_tile, cout, H, W):
    for sparse in (True, False):
        desc = ss.make_desc(cout, 24, 3, 3, wl.F16, wl.K_RSC)
        gen = torch.Generator(device="cuda").manual_seed(cout)
        rand = lambda *shape: torch.randn(shape, device="cuda", generator=gen)
        M = torch.tensor([1, 0, 0, 1], dtype=torch.uint8, device="cuda").repeat(cout, 54)
        w = (ss.ss_mask_compress if sparse else ss.ss_dense_pack)(desc, (rand(cout, 216) * 0.1).half(), M)
        x, res, bias = rand(1, H, W, 24).half(), rand(1, H, W, cout).half(), rand(cout)
        out = []
        for tile in (None, 2):
            force_tile(tile)
            out.append((ss.ss_conv2d_res_fwd if sparse else ss.ss_conv2d_dense_res_fwd)(desc, x, w, bias, res, (1, 1), (1, 1), wl.ACT_RELU))
        assert torch.isfinite(out[0]).all() and torch.equal(out[0].view(torch.int16), out[1].view(torch.int16)), sparse
