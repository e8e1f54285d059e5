"""The tiles of 96, 160 and 224 output channels (tile ids 6 to 8), whose 3, 5 or 7 waves are not a power of two: channel counts around the
tiles' edges and several tiles high, every staging mode that has them, with and without a residual, 16- and 8-bit operands.  (Dense FP8 has the 96 rows
channels-last only: its other combinations here run through the library's own choice.)"""
import pytest

import test_gpu_f8 as f8
import test_gpu_q8 as q8
import test_gpu_tail as tail
from helpers import check_close, oracle_ref, run_gpu
from paper_2411_00288_amd import workloads as wl

pytestmark = pytest.mark.gpu

ROWS = {6: 96, 7: 160, 8: 224}
# staging: (cin, flattening); K of the channels-last layers below and above a step's multiple
MODES = {"taps": (64, wl.K_CRS), "taps_ragged": (44, wl.K_CRS), "channels_last": (24, wl.K_RSC), "channels_last_long": (72, wl.K_RSC)}


def _couts(tile):
    b = ROWS[tile]
    return [b - 31, b, b + 1, 2 * b + 6]


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("tile", ROWS)
def test_sixteen_bit(ss, force_tile, tile, mode):
    cin, korder = MODES[mode]
    force_tile(tile)
    for i, cout in enumerate(_couts(tile)):
        dtype, act = (wl.F16, wl.BF16)[i % 2], (wl.ACT_RELU, wl.ACT_NONE, wl.ACT_GELU)[i % 3]
        L = tail._L(2, 9, 11, cin, cout, 3, s=1 + i // 3, p=1, dtype=dtype, korder=korder, act=act, seed=10 * tile + i)
        d = wl.make_inputs(L)
        ref, res = oracle_ref(L, d), tail._residual(L, i)
        ref_res = tail._ref(L, d, res)
        for sparse in (True, False):
            check_close(run_gpu(ss, L, d, sparse=sparse), ref, f"{L.name} tile {tile} sparse {sparse}")
            check_close(tail._run(ss, L, d, res, sparse=sparse), ref_res, f"{L.name} tile {tile} sparse {sparse} with a residual")


@pytest.mark.parametrize("cin,korder", [(64, wl.K_CRS), (48, wl.K_RSC), (128, wl.K_RSC)])
@pytest.mark.parametrize("tile", ROWS)
def test_eight_bit(ss, force_tile, tile, cin, korder):
    force_tile(tile)
    for i, cout in enumerate(_couts(tile)):
        L = q8._L(2, 9, 11, cin, cout, 3, s=1 + i // 3, p=1, korder=korder, seed=10 * tile + i)
        d = wl.make_inputs_q8(L)
        F = f8._L(2, 9, 11, cin, cout, 3, s=1 + i // 3, p=1, korder=korder, seed=10 * tile + i)
        e = wl.make_inputs_f8(F)
        for sparse in (True, False):
            q8.check_q8(q8._run(ss, L, d, sparse=sparse), q8._ref(L, d), f"{L.name} tile {tile} sparse {sparse}")
            check_close(f8._run(ss, F, e, sparse=sparse), f8._ref(F, e), f"{F.name} tile {tile} sparse {sparse}")
