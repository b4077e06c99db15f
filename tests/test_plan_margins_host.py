"""Plans that the cost model has been fitted without - whole rounds of big tiles with smaller ones behind them, a last column tile
past n, 192 rows in more row tiles than 256 need - are taken only where they lead by more than the model errs on them (no GPU:
the planner alone, on products that have been measured both ways)."""
import ctypes as C

import pytest

from paper_2601_11589_amd import api
from test_gpu_layer_tiles import PARTIAL, RESID, SWIGLU, Plan


def plan(m, n, k, epi, row_kernel, layer):
    f = api.lib()._Z14laps_gemm_planiiiiimbb
    f.restype = Plan
    p = f(C.c_int(m), C.c_int(n), C.c_int(k), C.c_int(0), C.c_int(epi), C.c_size_t(256 << 20), C.c_bool(row_kernel), C.c_bool(layer))
    return p.cfg, p.split, p.rest


@pytest.mark.parametrize("shape,want", [
    # 256 x 160 tiles in 1.75 and 2 rounds: 402 us, and 414 with 128 x 128 behind whole rounds of 256 x 256; 432 and 440
    ((3396, 5120, 13824, RESID, False, False), (4, 1, 0)), ((4096, 5120, 13824, RESID, False, True), (4, 1, 0)),
    ((7178, 2560, 9728, RESID, False, False), (4, 1, 0)),          # 290 and 304
    ((5219, 4608, 3584, PARTIAL, True, True), (9, 1, 0)),          # 134 and 138
    ((1138, 2560, 9728, RESID, True, True), (4, 3, 0)),            # 65.5 and 69.8 on 192 x 128 in 2 slices
    ((768, 7168, 5120, PARTIAL, True, True), (3, 2, 0)),           # 70.6 and 71.8 un-split on 192 x 128
])
def test_plans_behind_on_the_chip_are_not_taken(shape, want):
    assert plan(*shape) == want


@pytest.mark.parametrize("shape,want", [
    ((1847, 55296, 5120, SWIGLU, False, True), (10, 1, 1)), ((1024, 37888, 3584, SWIGLU, False, True), (2, 1, 8)),
    ((700, 27648, 5120, SWIGLU, False, False), (2, 1, 8)), ((256, 37888, 3584, SWIGLU, False, True), (9, 1, 0)),
    ((1847, 4608, 3584, PARTIAL, True, True), (4, 1, 0)), ((768, 4096, 4096, RESID, True, True), (7, 2, 0))])
def test_plans_ahead_on_the_chip_are(shape, want):
    assert plan(*shape) == want
