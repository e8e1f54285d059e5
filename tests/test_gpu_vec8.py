"""Sparse 8-bit channels-last layers whose tile the library takes by the length of the reduction (choose_vec8_sparse): the choice against the 128-row
tile, at the edges of the channel ranges that move to 256 rows and at a last tile of one pixel."""
import pytest
import torch

import test_gpu_f8 as f8
import test_gpu_q8 as q8
from paper_2411_00288_amd import workloads as wl

pytestmark = pytest.mark.gpu

# (images, height, width, channels in and out, kernel): K = 648 in 2-byte units, three rounds of 256-row tiles, nearly or just full
LAYERS = [(1, 191, 257, 144, 225, 3), (1, 192, 256, 144, 256, 3), (1, 128, 192, 144, 449, 3), (1, 3, 8171, 144, 511, 3)]


@pytest.mark.parametrize("N,H,W,cin,cout,k", LAYERS)
def test_choice_against_128_rows(ss, force_tile, N, H, W, cin, cout, k):
    for mod, make, exact in ((q8, wl.make_inputs_q8, True), (f8, wl.make_inputs_f8, False)):
        L = mod._L(N, H, W, cin, cout, k, p=k // 2 if k == 3 else 0, korder=wl.K_RSC, seed=cout)
        d = make(L)
        force_tile(None)
        y = mod._run(ss, L, d, sparse=True)
        force_tile(2)
        ref = mod._run(ss, L, d, sparse=True)
        if exact:                                         # whole sums, the same epilogue
            assert torch.equal(y.view(torch.int16), ref.view(torch.int16)), L.name
        else:                                             # K / 2 = 648 products at most in another order: 648 x 2^-24 of the sum of magnitudes, about
            a, b = y.float(), ref.float()                 # sqrt(648) = 26 rms of the result; then one rounding to binary16 on each side
            assert torch.isfinite(b).all()
            bound = 2.0 ** -10 * b.abs() + 648 * 2.0 ** -24 * 26 * b.pow(2).mean().sqrt()
            assert ((a - b).abs() <= bound).all(), L.name
