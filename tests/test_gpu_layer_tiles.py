"""The GEMM launches called directly: the 320 x 256 tile that only layers take, the launch of a captured graph that chooses its
tile by the live rows, the tiles up to 128 rows with live rows told late, and padding rows; at the edges of the tiles' rows and
with K slices of an odd and an even number of slabs.  Against float64, with rows of NaN behind the operand and guard rows
behind the result."""
import ctypes as C
import os
import re

import pytest
import torch

from paper_2601_11589_amd import api

PARTIAL, RESID, SWIGLU = 0, 1, 2
TILE_320 = 10


# GemmPlan's fields in the order of its definition (all of them int)
_HEADER = open(os.path.join(os.path.dirname(api.__file__), "csrc", "laps_internal.h")).read()
_FIELDS = re.findall(r"^    int (\w+);", re.search(r"struct GemmPlan \{(.*?)\n\};", _HEADER, re.S).group(1), re.M)


class Plan(C.Structure):
    _fields_ = [(name, C.c_int) for name in _FIELDS]

    def __init__(self, cfg, split, k_per_split, epi, ws):
        super().__init__(cfg=cfg, split=split, k_per_split=k_per_split, epi=epi, ws=ws)


def layer_plan(m, n, k, epi, row_kernel):
    """The plan a layer's driver makes.  (The symbols called here carry their argument types: a changed signature is not found.)"""
    f = api.lib()._Z14laps_gemm_planiiiiimbb
    f.restype = Plan
    return f(C.c_int(m), C.c_int(n), C.c_int(k), C.c_int(0), C.c_int(epi), C.c_size_t(256 << 20), C.c_bool(row_kernel), C.c_bool(True))


def launch(plan, a, w, m, out, resid, act, live=None):
    p = lambda t: C.c_void_p(t.data_ptr() if t is not None else 0)
    rc = api.lib()._Z16laps_gemm_launchRK8GemmPlanPKtS3_iiiPfPKfPtPKiS9_bP12ihipStream_t(
        C.byref(plan), p(a), p(w), C.c_int(m), C.c_int(w.shape[0]), C.c_int(w.shape[1]), p(out), p(resid), p(act), None, p(live),
        C.c_bool(live is not None), C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0, api.lib().laps_last_error()


def test_wide_rows_are_planned_in_layers_only():
    """In a layer where 320 rows save a row tile; a product of its own is reported with 256 rows at most."""
    for m, n, k, epi in ((300, 55296, 5120, SWIGLU), (640, 55296, 5120, SWIGLU), (11104, 5120, 27648, RESID), (1280, 7168, 5120, PARTIAL)):
        assert layer_plan(m, n, k, epi, epi != SWIGLU).cfg == TILE_320, (m, n, k)
        out = (C.c_int32 * 7)()
        assert api.lib().laps_gemm_plan_info(C.c_int32(m), C.c_int32(n), C.c_int32(k), C.c_int32(0), C.c_int32(epi), out) == 0
        assert out[0] <= 256
    for m in (129, 256, 400, 512, 1000):      # no fewer row tiles, or most of the last one padding
        assert layer_plan(m, 55296, 5120, SWIGLU, False).cfg != TILE_320, m


def run(plan, m, n, k, live=None, rows=None):
    """Runs one product of `rows` checked rows (default all m) and compares it with float64."""
    rows = m if rows is None else rows
    g = torch.Generator(device="cuda").manual_seed(m * 31 + n + k + rows)
    a = torch.full((m + 7, k), float("nan"), dtype=torch.bfloat16, device="cuda")
    a[:rows].normal_(0, 1, generator=g)
    w = torch.empty((n, k), dtype=torch.bfloat16, device="cuda").normal_(0, 0.02, generator=g)
    want = a[:rows].double() @ w.double().T
    out = torch.full((plan.split * m + 7, n), 7.0, device="cuda")
    act = torch.full((m + 7, n // 2), 7.0, dtype=torch.bfloat16, device="cuda")
    resid = None
    if plan.epi == RESID:
        resid = torch.empty((m, n), device="cuda").normal_(0, 4, generator=g)
    launch(plan, a, w, m, out, resid, act, live)
    torch.cuda.synchronize()
    assert bool((out[plan.split * m:] == 7).all()) and bool((act[m:] == 7).all())
    if plan.epi == SWIGLU:
        gate, up = want.view(rows, n // 64, 2, 32).unbind(2)
        ref = (torch.nn.functional.silu(gate) * up).reshape(rows, n // 2)
        # one bf16 rounding (at most 2^-8 of the value) of fp32 sums of k products, std 0.02 sqrt(k), which take k / 32
        # roundings of 2^-24 in a random walk: six standard deviations are delta; silu' is below 1.1
        delta = 6 * 2.0 ** -24 * 0.02 * k / 4
        slack = (delta * (1.1 * up.abs() + gate.abs())).reshape(rows, n // 2) + 1e-6
        assert bool(((act[:rows].double() - ref).abs() <= ref.abs() * 2.0 ** -8 + slack).all())
        return
    got = out[:plan.split * m].view(plan.split, m, n)[:, :rows].double().sum(0)
    ref = want if resid is None else want + resid[:rows].double()
    if rows:
        assert float((got - ref).norm() / ref.norm()) < 2e-6       # fp32 sums of exact products
        assert float((got - ref).abs().max()) < 2e-5 * float(ref.abs().max())


@pytest.mark.gpu
@pytest.mark.parametrize("m", [1, 160, 319, 320, 321, 657])
@pytest.mark.parametrize("k,split", [(64, 1), (192, 1), (1024, 1), (448, 2), (1024, 4)])
def test_320_row_tile_matches_float64(m, k, split):
    for epi in (PARTIAL,) if split > 1 else (PARTIAL, RESID, SWIGLU):
        per = -(-(k // 64) // split) * 64
        run(Plan(TILE_320, split, per, epi, 1), m, 512, k)


# widths that 256 x 160, 224 and 192 divide and that they do not; which tile runs is test_every_tile_by_live_rows_is_chosen's
@pytest.mark.gpu
@pytest.mark.parametrize("n,epi", [(5120, PARTIAL), (5120, RESID), (7168, PARTIAL), (3584, RESID), (4608, PARTIAL), (27648, SWIGLU), (37888, SWIGLU)])
def test_tile_by_live_rows_matches_float64(n, epi):
    for m, k in ((640, 320), (1024, 2048)):
        for rows in (1, 130, 256, 300, 513, 640):
            run(Plan(2, 1, k, epi, 1), m, n, k, torch.tensor([rows], dtype=torch.int32, device="cuda"), rows)
        run(Plan(TILE_320, 1, k, epi, 1), m, n, k, torch.tensor([m + 9], dtype=torch.int32, device="cuda"))
        none = Plan(2, 1, k, epi, 1)
        out, act = torch.full((m, n), 7.0, device="cuda"), torch.full((m, n // 2), 7.0, dtype=torch.bfloat16, device="cuda")
        a, w = torch.zeros((m, k), dtype=torch.bfloat16, device="cuda"), torch.zeros((n, k), dtype=torch.bfloat16, device="cuda")
        launch(none, a, w, m, out, out if epi == RESID else None, act, torch.tensor([0], dtype=torch.int32, device="cuda"))
        assert bool((out == 7).all()) and bool((act == 7).all())

# Up to 64 rows on tiles of 64 rows, then 128, or two of 64 where 128 columns make at most 128 workgroups (not the 129 tiles of
# 16512 columns, nor 2 and more slices of 16384): edges of both, weights bypassing the caches (rows given as live) and through them
# (a product of its own), with live rows told late and K slices of one and several slabs
@pytest.mark.gpu
@pytest.mark.parametrize("cfg,n", [(0, 256), (0, 16384), (0, 16512), (5, 512), (1, 192)])
@pytest.mark.parametrize("m", [1, 16, 63, 64, 65, 97, 128])
def test_tiles_up_to_128_rows_match_float64(cfg, n, m):
    for k, split in ((64, 1), (192, 1), (1024, 1), (448, 2), (1024, 4)):
        per = -(-(k // 64) // split) * 64
        for epi in (PARTIAL,) if split > 1 else (PARTIAL, RESID) + ((SWIGLU,) if cfg != 1 else ()):
            run(Plan(cfg, split, per, epi, 1), m, n, k)
            for rows in {1, (m + 1) // 2, m}:
                run(Plan(cfg, split, per, epi, 1), m, n, k, torch.tensor([rows], dtype=torch.int32, device="cuda"), rows)


@pytest.mark.gpu
@pytest.mark.parametrize("cfg,m,n", [(0, 100, 256), (5, 40, 512), (2, 300, 512), (10, 320, 512)])
def test_padding_rows_between_sequences_are_left_out(cfg, m, n):
    """Rows that row_live marks as padding hold NaN: they reach no other row, and a row tile of padding only is not written."""
    k = 320
    g = torch.Generator(device="cuda").manual_seed(m)
    live = torch.rand(m, device="cuda", generator=g) < 0.6
    live[256:] = False
    a = torch.empty((m, k), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)
    a[~live] = float("nan")
    w = torch.empty((n, k), dtype=torch.bfloat16, device="cuda").normal_(0, 0.02, generator=g)
    out = torch.full((m, n), 7.0, device="cuda")
    flags = torch.where(live, 3, -1).to(torch.int32)
    p = lambda t: C.c_void_p(t.data_ptr())
    assert api.lib()._Z16laps_gemm_launchRK8GemmPlanPKtS3_iiiPfPKfPtPKiS9_bP12ihipStream_t(
        C.byref(Plan(cfg, 1, k, PARTIAL, 1)), p(a), p(w), C.c_int(m), C.c_int(n), C.c_int(k), p(out), None, None, p(flags), None,
        C.c_bool(False), C.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    want = a[live].double() @ w.double().T
    assert float((out[live].double() - want).norm() / want.norm()) < 2e-6
    if cfg == 2:
        assert bool((out[256:] == 7).all())


def test_ragged_columns_are_planned_in_layers_only():
    """A last column tile past n where it fills the chip better; a product of its own keeps to widths that divide n."""
    for m, n, k, epi, cfg in ((256, 37888, 3584, SWIGLU, 9), (2776, 5120, 27648, RESID, 3), (1847, 4608, 3584, PARTIAL, 4)):
        p = layer_plan(m, n, k, epi, epi != SWIGLU)
        assert p.cfg == cfg and p.split == 1, (m, n, k, p.cfg, p.split)
        out = (C.c_int32 * 7)()
        assert api.lib().laps_gemm_plan_info(C.c_int32(m), C.c_int32(n), C.c_int32(k), C.c_int32(0), C.c_int32(epi), out) == 0
        assert n % out[1] == 0
    f = api.lib()._Z14laps_gemm_planiiiiimbb      # and never where 32-bit offsets do not reach
    f.restype = Plan
    for n in (192, 320, 640):
        p = f(C.c_int(700), C.c_int(n), C.c_int(1 << 22), C.c_int(0), C.c_int(PARTIAL), C.c_size_t(256 << 20), C.c_bool(True), C.c_bool(True))
        assert p.cfg in (1, 6, 7) and n % {1: 64, 6: 256, 7: 128}[p.cfg] == 0


# tile index -> columns; the last column tile holds 64 columns, all but 64, and (two and a bit) a whole one and 64
WIDTHS = {0: 128, 2: 256, 3: 224, 4: 160, 6: 256, 7: 128, 8: 128, 9: 192}


@pytest.mark.gpu
@pytest.mark.parametrize("cfg", sorted(WIDTHS))
@pytest.mark.parametrize("m", [129, 300])
def test_last_column_tile_past_n_matches_float64(cfg, m):
    width = WIDTHS[cfg]
    for n in sorted({64, -(-width // 64) * 64 - 64, -(-width // 64) * 64 + 64, 2 * width // 64 * 64 + 64}):
        if n % width == 0:
            continue
        for k, split in ((64, 1), (192, 1), (1024, 1), (448, 2), (1024, 4)):
            for epi in (PARTIAL,) if split > 1 else (PARTIAL, RESID) + ((SWIGLU,) if cfg not in (3, 4) else ()):
                run(Plan(cfg, split, -(-(k // 64) // split) * 64, epi, 1), m, n, k)


@pytest.mark.gpu
@pytest.mark.parametrize("n,epi", [(5120, RESID), (3584, RESID), (4608, PARTIAL), (27648, SWIGLU)])
def test_tile_by_live_rows_of_large_batches_matches_float64(n, epi):
    for rows in (1111, 1847, 2776, 3000):
        run(Plan(2, 1, 1024, epi, 1), 3000, n, 1024, torch.tensor([rows], dtype=torch.int32, device="cuda"), rows)


# whole rounds of big tiles and the columns behind them in smaller ones
def mixed(cfg, rest, k, epi):
    p = Plan(cfg, 1, k, epi, 1)
    p.rest = 1 + rest
    return p


def test_columns_behind_whole_rounds_are_planned_in_smaller_tiles():
    for m, n, k, epi, cfg, rest in ((1847, 55296, 5120, SWIGLU, 10, 0), (1024, 37888, 3584, SWIGLU, 2, 7), (1200, 55296, 5120, SWIGLU, 10, 8)):
        p = layer_plan(m, n, k, epi, epi != SWIGLU)
        assert (p.cfg, p.split, p.rest) == (cfg, 1, 1 + rest), (m, n, k, p.cfg, p.rest)
    for m in range(129, 5000, 53):       # whatever is planned fits: big tiles fill rounds, the others make at most one
        for n, k, epi in ((55296, 5120, SWIGLU), (27648, 5120, SWIGLU), (37888, 3584, SWIGLU), (5120, 27648, RESID), (7168, 5120, PARTIAL)):
            p = layer_plan(m, n, k, epi, epi != SWIGLU)
            if p.rest == 0:
                continue
            rows = {0: 128, 7: 192, 8: 256}[p.rest - 1]
            tiles_m = -(-m // {2: 256, 10: 320}[p.cfg])
            columns = tiles_m * (n // 256) // 256 * 256 // tiles_m
            assert p.split == 1 and 1 <= columns < n // 256 and -(-m // rows) * (n - columns * 256) // 128 <= 256, (m, n, p.cfg, p.rest)
    assert layer_plan(70000, 256, 5120, PARTIAL, True).rest == 0      # more row tiles than a round holds


@pytest.mark.gpu
@pytest.mark.parametrize("cfg,m,n", [(2, 257, 33024), (2, 700, 22272), (10, 321, 33024), (10, 961, 16640), (2, 513, 22016)])
@pytest.mark.parametrize("rest", [0, 7, 8])
def test_columns_behind_whole_rounds_match_float64(cfg, m, n, rest):
    for k in (64, 192):
        for epi in (PARTIAL, RESID, SWIGLU):
            run(mixed(cfg, rest, k, epi), m, n, k)
    # fewer live rows than an un-captured launch was made for: rows of NaN behind them reach nothing
    k, g = 192, torch.Generator(device="cuda").manual_seed(m + n)
    w = torch.empty((n, k), dtype=torch.bfloat16, device="cuda").normal_(0, 0.02, generator=g)
    for rows in (1, m - 130, m):
        a = torch.full((m, k), float("nan"), dtype=torch.bfloat16, device="cuda")
        a[:rows].normal_(0, 1, generator=g)
        out, live = torch.full((m, n), 7.0, device="cuda"), torch.tensor([rows], dtype=torch.int32, device="cuda")
        p = lambda t: C.c_void_p(t.data_ptr())
        assert api.lib()._Z16laps_gemm_launchRK8GemmPlanPKtS3_iiiPfPKfPtPKiS9_bP12ihipStream_t(
            C.byref(mixed(cfg, rest, k, PARTIAL)), p(a), p(w), C.c_int(m), C.c_int(n), C.c_int(k), p(out), None, None, None, p(live),
            C.c_bool(False), C.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
        want = a[:rows].double() @ w.double().T
        assert float((out[:rows].double() - want).norm() / want.norm()) < 2e-6


# The tile that gemm_live_kernel gives a number of rows, from the cost table and margins it is compiled with
_GEMM = open(os.path.join(os.path.dirname(api.__file__), "csrc", "gemm.hip")).read()
_LIST = lambda name: [int(v) for v in re.search(name + r"\[kLiveTiles\] = \{([^}]*)\}", _GEMM).group(1).split(",")]
LIVE_ROWS, LIVE_COLS, LIVE_CFG = _LIST("kLiveRows"), _LIST("kLiveCols"), _LIST("cfg")
COST = [[float(v) for v in t.split(",")] for t in re.findall(r"^    \{(\d+, \d+, \d, [\d.]+, [\d.]+, [\d.]+)\}, +// \d+:", _GEMM, re.M)]
MARGIN = [float(re.search(name + r" = ([\d.]+)", _GEMM).group(1)) for name in ("kRaggedMargin", "kMore192Margin")]


def tile_by_live_rows(m, n, k, epi):
    """Index among the tiles, and how far the next one is behind."""
    costs = []
    for i in range(5 if epi == SWIGLU else 7):
        _, _, _, fill, slab, part = COST[LIVE_CFG[i]]
        tiles_m = -(-m // LIVE_ROWS[i])
        tiles = tiles_m * -(-n // LIVE_COLS[i])
        us = -(-tiles // 256) * (fill + slab * (k // 64) * (1 - part * max(0, 1 - tiles / 256)))
        costs.append(us * (MARGIN[0] if n % LIVE_COLS[i] else MARGIN[1] if LIVE_ROWS[i] == 192 and tiles_m != -(-m // 256) else 1))
    best = sorted(costs)
    return costs.index(best[0]), best[1] / best[0]


# (rows, columns, K): tile, the last column tile past n or not; rows that fill no tile
LIVE = {(579, 16384, 192): (0, False), (257, 256, 192): (1, False), (257, 18944, 192): (2, True), (775, 8448, 192): (2, False),
        (257, 37888, 192): (3, False), (257, 27648, 192): (4, False), (390, 27648, 1024): (5, True), (1548, 7168, 192): (5, False),
        (257, 18944, 1024): (6, True), (3842, 2560, 320): (6, False)}
LIVE_CASES = [(c, epi) for c in LIVE for epi in (PARTIAL, RESID, SWIGLU) if epi != SWIGLU or LIVE[c][0] < 5]


def test_every_tile_by_live_rows_is_chosen():
    assert len(COST) == 11 and len(LIVE_ROWS) == len(LIVE_COLS) == len(LIVE_CFG) == 7
    assert all((LIVE_ROWS[i], LIVE_COLS[i]) == tuple(COST[LIVE_CFG[i]][:2]) for i in range(7))
    for epi in (PARTIAL, RESID, SWIGLU):
        seen = set()
        for case, e in LIVE_CASES:
            if e == epi:
                tile, lead = tile_by_live_rows(*case, epi)
                assert (tile, case[1] % LIVE_COLS[tile] != 0) == LIVE[case] and lead > 1.01, (case, epi)
                assert case[0] % LIVE_ROWS[tile] != 0
                seen.add(tile)
        assert seen == set(range(5 if epi == SWIGLU else 7))


@pytest.mark.gpu
@pytest.mark.parametrize("case,epi", LIVE_CASES)
def test_every_tile_by_live_rows_matches_float64(case, epi):
    rows, n, k = case
    run(Plan(2, 1, k, epi, 1), rows + 61, n, k, torch.tensor([rows], dtype=torch.int32, device="cuda"), rows)


# Padding between the sequences (row_live), as a batch with lengths shorter than its row offsets has it
@pytest.mark.gpu
@pytest.mark.parametrize("cfg,rest,m,n", [(9, None, 300, 320), (3, None, 700, 640), (4, None, 513, 448), (0, None, 300, 192), (7, None, 500, 320),
                                          (2, 0, 700, 22272), (2, 7, 513, 22016), (10, 8, 961, 16640), (10, 0, 1300, 16640)])
def test_padding_between_sequences_on_ragged_and_mixed_tiles(cfg, rest, m, n):
    k = 320
    g = torch.Generator(device="cuda").manual_seed(m + n)
    live = torch.rand(m, device="cuda", generator=g) < 0.6
    live[256:640] = False       # whole row tiles of every height
    live[m - 1] = True
    a = torch.empty((m, k), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)
    a[~live] = float("nan")
    w = torch.empty((n, k), dtype=torch.bfloat16, device="cuda").normal_(0, 0.02, generator=g)
    flags = torch.where(live, 3, -1).to(torch.int32)
    resid = torch.empty((m, n), device="cuda").normal_(0, 4, generator=g)
    want = a[live].double() @ w.double().T
    p = lambda t: C.c_void_p(t.data_ptr())
    for epi in (PARTIAL, RESID) + ((SWIGLU,) if cfg not in (3, 4) else ()):
        plan = Plan(cfg, 1, k, epi, 1) if rest is None else mixed(cfg, rest, k, epi)
        out = torch.full((m + 7, n), 7.0, device="cuda")
        act = torch.full((m + 7, n // 2), 7.0, dtype=torch.bfloat16, device="cuda")
        assert api.lib()._Z16laps_gemm_launchRK8GemmPlanPKtS3_iiiPfPKfPtPKiS9_bP12ihipStream_t(
            C.byref(plan), p(a), p(w), C.c_int(m), C.c_int(n), C.c_int(k), p(out), p(resid), p(act), p(flags), None, C.c_bool(False),
            C.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0, api.lib().laps_last_error()
        torch.cuda.synchronize()
        assert bool((out[m:] == 7).all()) and bool((act[m:] == 7).all())
        if epi == SWIGLU:      # bounds as in run()
            gate, up = want.view(-1, n // 64, 2, 32).unbind(2)
            ref = (torch.nn.functional.silu(gate) * up).reshape(-1, n // 2)
            slack = (6 * 2.0 ** -24 * 0.02 * k / 4 * (1.1 * up.abs() + gate.abs())).reshape(-1, n // 2) + 1e-6
            assert bool(((act[:m][live].double() - ref).abs() <= ref.abs() * 2.0 ** -8 + slack).all())
        else:
            ref = want if epi == PARTIAL else want + resid[live].double()
            assert float((out[:m][live].double() - ref).norm() / ref.norm()) < 2e-6
