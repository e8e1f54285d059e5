"""The tile of sparse 8-bit channels-last layers by channels and reduction (choose_vec8_sparse), on the host: both sides of its lines."""
import shutil
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parent.parent
LARGE = 64 * 256 * 40                               # forty tiles of pixels per compute unit: rounding plays no part


def test_both_sides(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    exe = tmp_path / "choose_vec8"
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", str(ROOT / "include"),
                    str(ROOT / "tests" / "host" / "choose_vec8.cpp"), "-o", str(exe)], check=True, capture_output=True)
    # (choice before, channels, reduction): 256 rows cost 1.53 + 118.4 / K, so the line of 0.86 lies at K = 623 for one tile against two
    want = {(2, 256, 620): 2, (2, 256, 626): 3, (2, 256, 2304): 3, (2, 225, 1024): 3, (2, 128, 2304): 2, (6, 96, 2304): 6, (2, 511, 1024): 3, (2, 449, 1024): 3,
            (8, 224, 2304): 8, (8, 448, 2304): 8, (2, 384, 2304): 2, (7, 160, 576): 7, (4, 256, 2304): 4, (5, 256, 2304): 5}
    lines = "".join(f"{id} {cout} {LARGE} {K}\n" for id, cout, K in want)
    out = subprocess.run([str(exe)], input=lines, capture_output=True, text=True, check=True).stdout.split()
    assert [int(o) for o in out] == list(want.values())


def test_rounds_of_the_grid(tmp_path):
    """Three rounds of 256-row tiles against six of 128 rows; one workgroup more and it is four against seven."""
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    exe = tmp_path / "choose_vec8"
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", str(ROOT / "include"),
                    str(ROOT / "tests" / "host" / "choose_vec8.cpp"), "-o", str(exe)], check=True, capture_output=True)
    want = {(2, 256, 64 * 768, 720): 3, (2, 256, 64 * 768 + 1, 720): 2, (2, 449, 64 * 384, 720): 3, (2, 449, 64 * 384 + 1, 720): 2}
    out = subprocess.run([str(exe)], input="".join("%d %d %d %d\n" % k for k in want), capture_output=True, text=True, check=True).stdout.split()
    assert [int(o) for o in out] == list(want.values())
