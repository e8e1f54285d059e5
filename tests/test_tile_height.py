"""The height of the tile by the output channels (choose_height), on the host: both sides of its lines."""
import shutil
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parent.parent
LARGE = 64 * 256 * 40                               # forty tiles of pixels per compute unit: rounding plays no part
S16, D16, S8, D8 = (0, 1), (0, 0), (1, 1), (1, 0)   # (bytes, sparse)


@pytest.fixture(scope="module")
def choose(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    exe = tmp_path_factory.mktemp("host") / "choose_height"
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", str(ROOT / "include"),
                    str(ROOT / "tests" / "host" / "choose_height.cpp"), "-o", str(exe)], check=True, capture_output=True)
    def run(id, cout, P, taps, form):
        out = subprocess.run([str(exe)], input=f"{id} {cout} {P} {taps} {form[0]} {form[1]}\n", capture_output=True, text=True, check=True)
        return int(out.stdout)
    return run


@pytest.mark.parametrize("cout,form,tile", [
    (65, S16, 6), (96, S16, 6), (97, S16, 2), (128, S16, 2), (129, S16, 7), (160, S16, 7), (161, S16, 8), (224, S16, 8), (225, S16, 3), (256, S16, 3), (256, D16, 2),
    (257, S16, 6), (288, S16, 6), (289, S16, 7), (320, S16, 7), (321, S16, 2), (384, S16, 2), (385, S16, 8), (448, S16, 8), (449, S16, 3), (449, D16, 2),
    (160, S8, 7), (160, D8, 7), (161, D8, 8), (288, D8, 6), (320, D8, 2), (400, D8, 8),
])
def test_large_grids(choose, cout, form, tile):
    assert choose(2, cout, LARGE, 1, form) == tile
    assert choose(3, cout, LARGE, 1, form) == tile           # (the paper's flattening compares all heights)


def test_the_channels_last_choice_between_128_and_256_rows_stands(choose):
    assert choose(2, 256, LARGE, 0, S16) == 2 and choose(3, 256, LARGE, 0, S16) == 3
    assert choose(2, 160, LARGE, 0, S16) == 7 and choose(3, 160, LARGE, 0, S16) == 7


def test_tiles_of_the_fullest_compute_unit_count(choose):
    """136 channels on 258 pixel tiles (two per compute unit on a few): still the 160-row tile, which halves the workgroups; 97 to 128
    channels never leave the 128-row one."""
    assert choose(2, 136, 64 * 258, 1, S16) == 7
    assert choose(2, 128, 64 * 258, 1, S16) == 2
    for id in (0, 1, 4, 5):                          # grids of one workgroup per unit and less, and the dense channels-last rule, keep theirs
        assert choose(id, 136, LARGE, 1, S16) == id


def test_dense_fp8_has_costs_of_its_own(tmp_path):
    """160 and 224 rows never; 96 rows channels-last only; in the paper's flattening 256 rows (with producer waves) by the length of the reduction."""
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    exe = tmp_path / "choose_height_f8"
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", str(ROOT / "include"),
                    str(ROOT / "tests" / "host" / "choose_height_f8.cpp"), "-o", str(exe)], check=True, capture_output=True)
    # (cout, taps, reduction steps): 9 to a chunk
    want = {(96, 1, 72): 2, (128, 1, 9): 2, (129, 1, 9): 2, (256, 1, 9): 2, (129, 1, 18): 3, (256, 1, 18): 3, (257, 1, 27): 2, (384, 1, 27): 2, (257, 1, 36): 3,
            (385, 1, 18): 3, (640, 1, 72): 3, (640, 1, 9): 2,
            (96, 0, 18): 6, (97, 0, 18): 2, (128, 0, 72): 2, (129, 0, 18): 6, (192, 0, 72): 6, (193, 0, 18): 2, (256, 0, 72): 2, (288, 0, 18): 6, (289, 0, 18): 2}
    lines = "".join(f"{2} {cout} {LARGE} {taps} {steps}\n" for cout, taps, steps in want)
    out = subprocess.run([str(exe)], input=lines, capture_output=True, text=True, check=True).stdout.split()
    assert [int(o) for o in out] == list(want.values())
