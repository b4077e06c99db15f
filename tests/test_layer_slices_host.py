"""K slices of a layer's projections up to 128 rows (no GPU: the planner alone): whatever follows the product, its partial sums fit
the region that a workspace of its rows or of more lays out for them, its workgroups fit one round of the compute units, the slices
cover K with none empty, and all but the last hold at least 6 slabs of 64 (8 are asked for, in a whole number of slices)."""
import ctypes as C

import pytest

from paper_2601_11589_amd import api, inputs

ROWS = (1, 8, 63, 64, 65, 72, 79, 80, 95, 96, 112, 128)
BIG = 256 << 20


class Plan(C.Structure):
    _fields_ = [(f, C.c_int) for f in ("cfg", "split", "k_per_split", "epi", "ws", "rest")]


def layer_plan(m, n, k, epi, follows):
    f = api.lib()._Z14laps_gemm_planiiiiimbb
    f.restype = Plan
    return f(C.c_int(m), C.c_int(n), C.c_int(k), C.c_int(0), C.c_int(epi), C.c_size_t(BIG), C.c_bool(follows), C.c_bool(True))


@pytest.mark.parametrize("n,k", [(7168, 5120), (5120, 5120), (5120, 13824), (5120, 27648), (4608, 3584), (3584, 3584), (3584, 18944),
                                 (6144, 4096), (5120, 4096), (2048, 2048), (1536, 1536), (768, 256), (256, 256), (256, 704), (192, 256),
                                 (1024, 4672)])
def test_slices_of_layer_products(n, k):
    tile = api.lib()._Z19laps_gemm_tile_dimsiPiS_
    for m in ROWS:
        for epi in (0, 1, 2):
            for follows in (False, True):
                p = layer_plan(m, n, k, epi, follows)
                bm, bn = C.c_int(), C.c_int()
                tile(p.cfg, C.byref(bm), C.byref(bn))
                assert p.split >= 1 and (p.split - 1) * p.k_per_split < k <= p.split * p.k_per_split
                last = (k - (p.split - 1) * p.k_per_split) // 64        # the rest, of one slab where 73 are cut into nine
                assert last >= p.ws and last % p.ws == 0
                assert p.split * -(-n // bn.value) <= 256
                assert p.split == 1 or p.k_per_split >= 6 * 64


def partial_region(cfg, rows, seqs):
    """What a workspace holds behind everything else, from its total and the layout's other regions."""
    c = api._ModelCfg(cfg.hidden, cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, cfg.intermediate, 1, 16, 0, 1e6, 1e-6)
    table = api.lib()._Z26laps_attn_item_table_bytesiii
    table.restype = C.c_size_t
    qd = cfg.n_q_heads * cfg.head_dim
    up = lambda b: (b + 255) // 256 * 256
    rest = (2 * up(rows * 4) + up(seqs * 4) + up((seqs + 1) * 4) + up(table(C.c_int(rows), C.c_int(seqs), C.c_int(cfg.n_q_heads // cfg.n_kv_heads)))
            + up(rows * cfg.hidden * 2) + 2 * up(rows * qd * 2) + up(rows * cfg.intermediate * 2) + up(rows * cfg.hidden * 4))
    return api.lib().laps_workspace_bytes_for(C.byref(c), C.c_int32(rows), C.c_int32(seqs)) - rest


@pytest.mark.parametrize("cfgf", [inputs.tiny_cfg, inputs.qwen7b_cfg, inputs.qwen14b_cfg, inputs.qwen32b_cfg])
def test_partial_sums_fit_the_workspace(cfgf):
    cfg = cfgf(1)
    d, qd, inter = cfg.hidden, cfg.n_q_heads * cfg.head_dim, cfg.intermediate
    qkv = qd + 2 * cfg.n_kv_heads * cfg.head_dim
    for m in range(1, 129):
        rooms = [partial_region(cfg, rows, min(rows, 4)) for rows in {m, 128, 200, 1024}]
        for n, k, epi, follows in ((qkv, d, 0, True), (d, qd, 1, True), (2 * inter, d, 2, False), (d, inter, 1, True), (d, inter, 1, False)):
            p = layer_plan(m, n, k, epi, follows)
            if p.epi == 0:      # raw sums, of one slice too
                assert p.split * m * n * 4 <= min(rooms), (m, n, k, p.split)


@pytest.mark.parametrize("m,n,k,epi,split", [
    (128, 5120, 5120, 1, 5), (96, 5120, 5120, 1, 5),               # 24.8 and 21.9 us in 5 slices, 25.1 and 22.3 in 6
    (8, 5120, 4096, 1, 4), (64, 5376, 4096, 1, 4),                 # 16 slabs in slices of 12: 13.4 and 14.1; 17.7 and 18.3
    (72, 4352, 4096, 1, 4), (96, 4096, 6144, 1, 6),                # 16.7 and 17.3 in 7; 20.8 and 21.7 in 8
    (72, 3584, 5120, 0, 8), (96, 3584, 5120, 0, 4),                # pairs of 64 rows in half the slices 17.6 against 17.0, 18.8 against 19.4
    (8, 3584, 3584, 1, 7), (8, 2048, 2048, 1, 4), (128, 2048, 2048, 1, 4), (128, 4608, 3584, 0, 3)])
def test_slices_are_those_that_measured_faster(m, n, k, epi, split):
    assert layer_plan(m, n, k, epi, True).split == split
