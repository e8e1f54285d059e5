"""Which kernel an inverted bottleneck takes (choose_mlp), on the host: both sides of each line."""
import shutil
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parent.parent
RELU, GELU = 1, 2


def test_both_sides_of_the_lines(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    exe = tmp_path / "choose_mlp"
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", str(ROOT / "include"),
                    str(ROOT / "tests" / "host" / "choose_mlp.cpp"), "-o", str(exe)], check=True, capture_output=True)
    few, six, twelve = 32 * 256, 6 * 32 * 256, 12 * 32 * 256      # the last pixels of one workgroup, of six and of twelve tiles per compute unit
    # (pixels, input, intermediate, output channels, first activation, sparse): kernel, can the resident one run it
    want = {}
    for sparse in (0, 1):
        want.update({(few, 64, 256, 64, GELU, sparse): (41, 0), (few + 1, 64, 256, 64, GELU, sparse): (40, 0), (few, 32, 128, 32, GELU, sparse): (40, 0),
                     (few, 64, 512, 32, GELU, sparse): (41, 0), (few, 64, 640, 64, GELU, sparse): (40, 0), (few, 32, 256, 32, GELU, sparse): (41, 0),
                     (few, 32, 256, 32, RELU, sparse): (40, 0), (few, 64, 256, 32, RELU, sparse): (40, 0), (few, 64, 256, 64, RELU, sparse): (41, 0),
                     (few, 32, 256, 96, RELU, sparse): (41, 0), (six, 96, 384, 96, RELU, sparse): (40, 1), (six + 1, 96, 384, 96, RELU, sparse): (42, 1),
                     (six + 1, 96, 384, 96, 0, sparse): (42, 1), (six + 1, 96, 384, 128, RELU, sparse): (40, 0), (six + 1, 64, 256, 64, RELU, sparse): (40, 0),
                     (six + 1, 96, 512, 96, RELU, sparse): (42 if sparse else 40, sparse), (six + 1, 96, 640, 96, RELU, sparse): (42 if sparse else 40, sparse),
                     (six + 1, 96, 768, 96, RELU, sparse): (40, 0), (six + 1, 96, 384, 96, GELU, sparse): (40 if sparse else 42, 1 - sparse)})
        # 128 channels: sparse only, later for short intermediates, never for the shortest
        for cmid, line in ((128, None), (256, twelve), (384, twelve), (512, six)):
            for P in (six, six + 1, twelve, twelve + 1):
                want[(P, 128, cmid, 128, RELU, sparse)] = (42 if sparse and line is not None and P > line else 40, sparse)
        want[(twelve + 1, 128, 640, 128, RELU, sparse)] = (40, 0)
    out = subprocess.run([str(exe)], input="".join("%d %d %d %d %d %d\n" % k for k in want), capture_output=True, text=True, check=True).stdout.split()
    assert [(int(a), int(b)) for a, b in zip(out[::2], out[1::2])] == list(want.values())
