"""The tile choice for channels-last layers with taps on large grids (choose_vec), on the host: both sides of every line of the rule."""
import shutil
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parent.parent
LARGE = 50176                                       # pixels: 64 images of 28x28
S16, D16, S8, D8 = (0, 1), (0, 0), (1, 1), (1, 0)   # (bytes, sparse)


@pytest.fixture(scope="module")
def choose(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    exe = tmp_path_factory.mktemp("host") / "choose_vec"
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", str(ROOT / "include"),
                    str(ROOT / "tests" / "host" / "choose_vec.cpp"), "-o", str(exe)], check=True, capture_output=True)
    def run(cout, K, P, form):
        out = subprocess.run([str(exe)], input=f"{cout} {K} {P} {form[0]} {form[1]}\n", capture_output=True, text=True, check=True)
        return int(out.stdout)
    return run


@pytest.mark.parametrize("cout,K,P,form,tile", [
    # sparse 16-bit: tiles of the fullest of 256 compute units, two of 128 rows against 9/8 of one of 256
    (256, 2304, LARGE, S16, 2), (256, 2304, 98000, S16, 3),                             # 7 : 4 and 12 : 6
    (257, 576, LARGE, S16, 2), (384, 2304, LARGE, S16, 2), (385, 2304, LARGE, S16, 3),  # 10 : 7, 13 : 7
    (512, 576, 21560, S16, 3), (576, 2304, LARGE, S16, 2), (640, 576, LARGE, S16, 2), (641, 576, LARGE, S16, 3), (1024, 2304, LARGE, S16, 3),
    # dense 16-bit: 128 rows while they are fewer, or the reduction is short; producer waves otherwise
    (256, 1791, LARGE, D16, 2), (256, 1792, LARGE, D16, 5), (320, 4608, LARGE, D16, 2), (385, 1792, LARGE, D16, 5), (512, 1152, LARGE, D16, 2),
    (512, 2304, LARGE, D16, 5), (800, 2304, LARGE, D16, 2), (1024, 2304, LARGE, D16, 5),
    # dense 8-bit: 128 rows; sparse 8-bit: up to 512 channels
    (256, 2304, LARGE, D8, 2), (512, 576, LARGE, D8, 2), (320, 1152, LARGE, S8, 2), (511, 2304, LARGE, S8, 2), (512, 2304, LARGE, S8, 3),
])
def test_large_grids(choose, cout, K, P, form, tile):
    assert choose(cout, K, P, form) == tile


@pytest.mark.parametrize("form", [S16, D16, S8, D8])
def test_other_grids_keep_the_general_choice(choose, form):
    assert choose(256, 2304, 64 * 255, form) == 5         # one 256-row tile per compute unit: producer waves
    assert choose(128, 2304, 64 * 100, form) == 4
    assert choose(128, 2304, LARGE, form) == 2
    assert choose(256, 2304, 64 * 300, form) == 2         # below 512 tiles of 256 rows
    assert choose(64, 2304, 64 * 100, form) == 1
