"""Which kernel a depthwise layer takes (choose_dw), on the host: both sides of each line."""
import shutil
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parent.parent


def _choices(tmp_path, shapes):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    exe = tmp_path / "choose_dw"
    subprocess.run(["g++", "-std=c++17", "-O1", str(ROOT / "tests" / "host" / "choose_dw.cpp"), "-o", str(exe)], check=True, capture_output=True)
    out = subprocess.run([str(exe)], input="".join("%d %d %d %d %d %d\n" % s for s in shapes), capture_output=True, text=True, check=True).stdout.split()
    return [int(o) for o in out]


def test_layers_that_a_kernel_cannot_number_go_to_the_vector_kernel(tmp_path):
    """Outputs of more threads than the kernel for few outputs can number, and rows too long for its offsets: another kernel, no refusal."""
    want = {(4, 3, 1, 8, 3, 1 << 29): 60, (2, 3, 1, 8, 3, 1 << 28): 65, (1, 64, 200000, 896, 3, 1): 60, (1, 64, 190000, 896, 3, 1): 65, (1, 30, 30, 912, 3, 1): 60}
    assert _choices(tmp_path, want) == list(want.values())


def test_both_sides_of_the_lines(tmp_path):
    want = {}
    for k, rows in ((3, {1: ((26041, 63), (26042, 60)), 2: ((13020, 63), (13021, 64), (41666, 64), (41667, 64)), 3: ((8680, 63), (8681, 64), (27777, 64), (27778, 65))}),
                    (5, {1: ((12499, 63), (12500, 60), (43690, 60), (43691, 61)), 2: ((13020, 63), (13021, 60)), 3: ((17361, 63), (17362, 61))})):
        for H, lines in rows.items():
            want.update({(N, H, 1, 96, k, k // 2): tile for N, tile in lines})
    # 5x5 with more than 128 channels; 7x7: 1.7 and 3.2 M outputs, pairs of columns while they are one workgroup per compute unit
    want.update({(10280, 3, 1, 136, 5, 2): 63, (10281, 3, 1, 136, 5, 2): 61, (1, 195, 14, 96, 7, 3): 62, (1, 196, 14, 96, 7, 3): 63, (5902, 3, 1, 96, 7, 3): 63,
                 (5903, 3, 1, 96, 7, 3): 64, (11111, 3, 1, 96, 7, 3): 64, (11112, 3, 1, 96, 7, 3): 61})
    assert _choices(tmp_path, want) == list(want.values())
