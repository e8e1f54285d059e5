"""Max pooling with its fixed-size windows: borders, strides, signed zeros in either order, NaNs and infinities, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2411_00288_amd import workloads as wl
from helpers import host_bits

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [wl.F16, wl.BF16])
@pytest.mark.parametrize("k,s,p,H,W", [(3, 2, 1, 13, 10), (3, 1, 1, 6, 7), (3, 3, 0, 7, 7), (2, 2, 0, 9, 6), (2, 1, 1, 5, 5), (4, 2, 2, 8, 9)])
def test_maxpool_special_values(ss, dtype, k, s, p, H, W):
    rng = np.random.Generator(np.random.PCG64(k * 100 + H))
    xb = wl.to_bits(rng.standard_normal((2, H, W, 24), dtype=np.float32), dtype)
    special = np.array([0x0000, 0x8000, 0x8000, 0x0000, 0x7F80 if dtype == wl.BF16 else 0x7C00, 0xFF80 if dtype == wl.BF16 else 0xFC00,
                        0x0001, 0x8001], dtype=np.uint16)
    zeros = rng.random(xb.shape) < 0.7                       # most windows hold nothing but zeros of both signs and negatives
    xb = np.where(zeros, rng.choice(special[:4], xb.shape), xb)
    xb = np.where(rng.random(xb.shape) < 0.05, rng.choice(special, xb.shape), xb).astype(np.uint16)
    xb[1] = np.where(rng.random(xb[1].shape) < 0.03, np.uint16(0x7FC1), xb[1])
    y = ss.ss_maxpool2d(torch.from_numpy(xb.view(np.int16)).cuda().view(torch.float16 if dtype == wl.F16 else torch.bfloat16), k, s, p)
    assert np.array_equal(host_bits(y), oracle.maxpool2d(xb, dtype=dtype, k=k, stride=s, pad=p))
