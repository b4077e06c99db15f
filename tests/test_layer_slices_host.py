"""K slices of a layer's projections up to 128 rows (no GPU: the planner alone): whatever follows the product, its partial sums
fit what the workspace reserves for them, its workgroups fit one round of the compute units, and a slice holds at least 8 slabs
of 64 where K is cut for a row kernel's sake."""
import ctypes as C

import pytest

from paper_2601_11589_amd import api

ROWS = (1, 8, 63, 64, 65, 72, 95, 96, 112, 128)
BIG = 256 << 20


class Plan(C.Structure):
    _fields_ = [(f, C.c_int) for f in ("cfg", "split", "k_per_split", "epi", "ws", "rest")]


@pytest.mark.parametrize("n,k", [(7168, 5120), (5120, 5120), (5120, 13824), (5120, 27648), (4608, 3584), (3584, 3584), (3584, 18944),
                                 (6144, 4096), (2048, 2048), (1536, 1536), (768, 256), (256, 256), (256, 704), (192, 256)])
def test_slices_of_layer_products(n, k):
    plan, room = api.lib()._Z14laps_gemm_planiiiiimbb, api.lib()._Z23laps_gemm_partial_bytesiiim
    plan.restype, room.restype = Plan, C.c_size_t
    tile = api.lib()._Z19laps_gemm_tile_dimsiPiS_
    for m in ROWS:
        have = room(m, n, k, C.c_size_t(BIG))
        for epi in (0, 1, 2):
            for follows in (False, True):
                p = plan(m, n, k, 0, epi, C.c_size_t(BIG), C.c_bool(follows), C.c_bool(True))
                bm, bn = C.c_int(), C.c_int()
                tile(p.cfg, C.byref(bm), C.byref(bn))
                assert p.split >= 1 and (p.split - 1) * p.k_per_split < k <= p.split * p.k_per_split
                assert p.split == 1 or p.split * m * n * 4 <= have
                assert p.split * -(-n // bn.value) <= 256
                assert p.split == 1 or p.k_per_split >= 6 * 64       # 8 slabs asked for, rounded up to even slices of at least 6
