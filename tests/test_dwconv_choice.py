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
