"""The GEMM tiles above 128 rows, at the edges of the row tiles and with K slices of an odd and an even number of
slabs, against float64; and, on the CPU, the bound that the partial sums of their K splits keep."""
import ctypes as C

import pytest
import torch

from paper_2601_11589_amd import api, inputs

PARTIAL, RESID, SWIGLU = 0, 1, 2


def plan(m, n, k, epi):
    out = (C.c_int32 * 7)()
    assert api.lib().laps_gemm_plan_info(C.c_int32(m), C.c_int32(n), C.c_int32(k), C.c_int32(0), C.c_int32(epi), out) == 0
    return dict(zip(("bm", "bn", "split", "k_per", "epi", "ws", "wgs"), list(out)))


@pytest.mark.parametrize("cfgf", [inputs.tiny_cfg, inputs.qwen7b_cfg, inputs.qwen14b_cfg, inputs.qwen32b_cfg])
def test_partial_sums_of_an_automatic_split_stay_within_their_bound(cfgf):
    """256 MiB, and no more than the workspace of a layer of these rows has room for."""
    c = cfgf(1)
    shapes = ((c.qkv_dim, c.hidden, PARTIAL), (c.hidden, c.q_dim, RESID), (2 * c.intermediate, c.hidden, SWIGLU),
              (c.hidden, c.intermediate, RESID))
    mc = api._ModelCfg(c.hidden, c.n_q_heads, c.n_kv_heads, c.head_dim, c.intermediate, 1, 16, 0, 1e6, 1e-6)
    for m in list(range(129, 800, 7)) + [1024, 1200, 1280, 2048, 4096, 12000]:
        room = api.lib().laps_workspace_bytes_for(C.byref(mc), C.c_int32(m), C.c_int32(1))
        for n, k, epi in shapes:
            p = plan(m, n, k, epi)
            assert p["split"] == 1 or p["split"] * m * n * 4 <= min(room, 256 << 20), (m, n, k, p)


@pytest.mark.parametrize("m,n,k,epi,slices", [(1200, 3584, 18944, RESID, 3), (1500, 3584, 18944, RESID, 3), (2048, 3584, 18944, RESID, 2),
                                              (640, 5120, 27648, RESID, 4), (1280, 5120, 27648, RESID, 5), (1400, 5120, 27648, RESID, 2),
                                              (2200, 5120, 27648, RESID, 4), (640, 4864, 7168, PARTIAL, 2), (1280, 3584, 11136, SWIGLU, 3)])
def test_k_is_split_where_tiles_leave_the_chip_idle(m, n, k, epi, slices):
    """Products whose fp32 partial sums are large but pay for themselves: fewer slices are slower, and sums of longer
    chains less precise."""
    assert plan(m, n, k, epi)["split"] >= slices


# Every tile with K slices of any number of slabs (odd K / 64) and of multiples of two, each epilogue it is built with and K splits
# (tile rows, columns, slabs that a K slice holds a multiple of, epilogue, split), and the smallest product of whole and ragged row tiles that is planned on it.
TILES = [
    (128, 128, 1, PARTIAL, True, 129, 128, 576), (128, 128, 1, PARTIAL, False, 129, 128, 192), (128, 128, 1, RESID, False, 129, 128, 192),
    (128, 128, 1, SWIGLU, False, 129, 128, 192), (128, 128, 2, PARTIAL, True, 129, 128, 512), (128, 128, 2, PARTIAL, False, 129, 128, 256),
    (128, 128, 2, RESID, False, 129, 128, 256), (128, 128, 2, SWIGLU, False, 129, 128, 256),
    (128, 64, 1, PARTIAL, True, 129, 192, 576), (128, 64, 1, PARTIAL, False, 129, 192, 192), (128, 64, 1, RESID, False, 129, 192, 192),
    (128, 64, 2, PARTIAL, True, 129, 192, 512), (128, 64, 2, PARTIAL, False, 129, 192, 256), (128, 64, 2, RESID, False, 129, 192, 256),
    (256, 256, 1, SWIGLU, True, 385, 6400, 6208), (256, 256, 1, PARTIAL, False, 900, 13824, 192), (256, 256, 1, RESID, False, 1537, 8192, 192),
    (256, 256, 1, SWIGLU, False, 900, 13824, 192), (256, 256, 2, SWIGLU, True, 385, 6400, 6144), (256, 256, 2, PARTIAL, False, 900, 13824, 256),
    (256, 256, 2, RESID, False, 1537, 8192, 256), (256, 256, 2, SWIGLU, False, 900, 13824, 256),
    (256, 224, 1, PARTIAL, True, 1537, 448, 10304), (256, 224, 1, PARTIAL, False, 1300, 7168, 320), (256, 224, 1, RESID, False, 1300, 7168, 320),
    (256, 224, 2, PARTIAL, True, 1537, 448, 10240), (256, 224, 2, PARTIAL, False, 1300, 7168, 384), (256, 224, 2, RESID, False, 1300, 7168, 384),
    (256, 160, 1, PARTIAL, True, 129, 2240, 8256), (256, 160, 1, PARTIAL, False, 1537, 5120, 192), (256, 160, 1, RESID, False, 1537, 5120, 192),
    (256, 160, 2, PARTIAL, True, 129, 2240, 8192), (256, 160, 2, PARTIAL, False, 1537, 5120, 256), (256, 160, 2, RESID, False, 1537, 5120, 256),
    (128, 256, 1, PARTIAL, True, 257, 6144, 2112), (128, 256, 1, PARTIAL, False, 1537, 2560, 192), (128, 256, 1, RESID, False, 1537, 2560, 192),
    (128, 256, 1, SWIGLU, False, 1537, 2560, 192), (128, 256, 2, PARTIAL, True, 257, 6144, 2560), (128, 256, 2, PARTIAL, False, 1537, 2560, 256),
    (128, 256, 2, RESID, False, 1537, 2560, 256), (128, 256, 2, SWIGLU, False, 1537, 2560, 256),
    (192, 256, 1, SWIGLU, True, 257, 6144, 6208), (192, 256, 1, PARTIAL, False, 513, 16384, 448), (192, 256, 1, SWIGLU, False, 513, 16384, 448),
    (192, 256, 2, PARTIAL, True, 257, 6144, 5120), (192, 256, 2, PARTIAL, False, 513, 16384, 512), (192, 256, 2, SWIGLU, False, 513, 16384, 512),
    (192, 128, 1, PARTIAL, True, 129, 6144, 1536), (192, 128, 1, PARTIAL, False, 257, 13824, 192), (192, 128, 1, RESID, False, 513, 7168, 192),
    (192, 128, 1, SWIGLU, False, 257, 13824, 192),
    (256, 128, 1, PARTIAL, True, 769, 2688, 2112), (256, 128, 1, PARTIAL, False, 1537, 2688, 192), (256, 128, 1, RESID, False, 1537, 2688, 192),
    (256, 128, 1, SWIGLU, False, 1537, 2688, 192), (256, 128, 2, PARTIAL, True, 385, 3072, 4096), (256, 128, 2, PARTIAL, False, 1537, 2688, 256),
    (256, 128, 2, RESID, False, 1537, 2688, 256), (256, 128, 2, SWIGLU, False, 1537, 2688, 256),
    (256, 192, 1, PARTIAL, True, 513, 1344, 6208), (256, 192, 1, PARTIAL, False, 513, 13824, 192), (256, 192, 1, RESID, False, 1300, 6144, 192),
    (256, 192, 1, SWIGLU, False, 513, 13824, 192), (256, 192, 2, PARTIAL, True, 1537, 1344, 1536), (256, 192, 2, PARTIAL, False, 513, 13824, 256),
    (256, 192, 2, RESID, False, 1300, 6144, 256), (256, 192, 2, SWIGLU, False, 513, 13824, 256)]


def test_every_tile_has_a_product():
    for bm, bn, ws, epi, split, m, n, k in TILES:
        p = plan(m, n, k, epi)
        assert (p["bm"], p["bn"], p["ws"], p["split"] > 1) == (bm, bn, ws, split), ((m, n, k, epi), p)
        assert p["epi"] == (PARTIAL if split else epi)


def operands(m, n, k):
    g = torch.Generator(device="cuda").manual_seed(m * 31 + n + k)
    a = torch.empty((m, k), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)
    w = torch.empty((n, k), dtype=torch.bfloat16, device="cuda").normal_(0, 0.02, generator=g)
    return g, a, w, a.double() @ w.double().T


def check_product(ctx, g, a, w, want, epi):
    (m, k), n = a.shape, w.shape[0]

    def rel(got, ref):
        return float((got.double() - ref).norm() / ref.norm())

    if epi == PARTIAL:
        assert rel(ctx.laps_gemm_bf16(a, w), want) < 2e-6          # fp32 sums of exact products
    elif epi == RESID:
        resid = torch.empty((m, n), device="cuda").normal_(0, 4, generator=g)
        assert rel(ctx.laps_gemm_epilogue_bf16(a, w, 1, resid=resid), resid.double() + want) < 2e-6
    else:
        gate, up = want.view(m, n // 64, 2, 32).unbind(2)            # gate and up columns interleaved in blocks of 32
        ref = (torch.nn.functional.silu(gate) * up).reshape(m, n // 2)
        got = ctx.laps_gemm_epilogue_bf16(a, w, 2).double()
        # One bf16 rounding (half an ulp is at most 2^-8 of the value) of fp32 sums and an fp32 SiLU.  A sum of k products,
        # std 0.02 sqrt(k), takes k / 16 roundings of 2^-24 in a random walk: six standard deviations are
        # delta = 6 * 2^-24 * 0.02 sqrt(k) * sqrt(k / 16); silu' is below 1.1, so the product moves by at most
        # delta * (1.1 |up| + |gate|).
        delta = 6 * 2.0 ** -24 * 0.02 * k / 4
        slack = (delta * (1.1 * up.abs() + gate.abs())).reshape(m, n // 2) + 1e-6
        assert bool(((got - ref).abs() <= ref.abs() * 2.0 ** -8 + slack).all())


@pytest.mark.gpu
@pytest.mark.parametrize("bm,bn,ws,epi,split,m,n,k", TILES)
def test_tile_matches_float64(bm, bn, ws, epi, split, m, n, k):
    ctx = api.LapsCtx(inputs.tiny_cfg(1), max_positions=64)
    check_product(ctx, *operands(m, n, k), epi)
    ctx.close()


# (rows, columns, K) at the edges of row tiles, each with every epilogue
SHAPES = [(129, 128, 64), (191, 256, 192), (257, 128, 1088), (255, 384, 128), (513, 8192, 64), (576, 8192, 128),
          (513, 3584, 1024), (576, 3584, 1088), (1025, 4096, 576), (1025, 4096, 512), (192, 27648, 5120),
          (300, 27648, 5120), (384, 5120, 13824), (700, 27648, 1024)]
# up to 128 rows, either side of the 48 rows above which the weights of split products come through the caches, and of a 16-row
# sub-tile
SHAPES += [(m, n, k) for n, k in ((5120, 5120), (5120, 13824), (4160, 5120)) for m in (16, 17, 48, 49, 128)]


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,k", SHAPES)
def test_tiles_above_128_rows_match_float64(m, n, k):
    ctx = api.LapsCtx(inputs.tiny_cfg(1), max_positions=64)
    product = operands(m, n, k)
    print("plan", plan(m, n, k, PARTIAL), plan(m, n, k, RESID), plan(m, n, k, SWIGLU), flush=True)
    check_product(ctx, *product, PARTIAL)
    if n <= 8192:
        check_product(ctx, *product, RESID)
    if n % 128 == 0:
        check_product(ctx, *product, SWIGLU)
    ctx.close()


@pytest.mark.parametrize("n", [64, 128, 256, 384])
@pytest.mark.parametrize("m", [1, 64, 130, 400])
@pytest.mark.parametrize("k", [1 << 22, (1 << 22) + 64])
def test_long_rows_fill_the_chip_and_keep_their_sums_short(m, n, k):
    """Rows of 2^22 values and more: the few tiles there are split K until they fill the chip, as shorter rows do."""
    for epi in (PARTIAL, RESID, SWIGLU):
        p = plan(m, n, k, epi)
        assert p["wgs"] >= 128 and p["k_per"] <= k // 16 and (p["split"] - 1) * p["k_per"] < k <= p["split"] * p["k_per"], p
        assert p["split"] * m * n * 4 <= 256 << 20, p


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,k", [(4, 128, (1 << 22) + 64), (130, 128, 1 << 22), (130, 64, 1 << 22), (130, 256, (1 << 22) - 128),
                                   (64, 256, 1 << 22), (200, 256, (1 << 22) + 64), (400, 128, 1 << 22),
                                   (700, 1024, (1 << 22) - 128), (600, 1280, (1 << 22) - 64)])
def test_rows_at_the_reach_of_32_bit_offsets(m, n, k):
    """Rows of 2^22 values and more are addressed by pointers, shorter ones by 32-bit offsets: on 256-row tiles the last
    rows of the last two shapes lie just below 2^31 bytes behind the tile's first.  Operands of -1, 0 and 1:
    every fp32 sum is a whole number below 2^24, hence exact."""
    if m >= 600:
        assert (plan(m, n, k, PARTIAL)["bm"], plan(m, n, k, PARTIAL)["bn"]) == (256, 256) == (plan(m, n, k, RESID)["bm"], plan(m, n, k, RESID)["bn"])
    ctx = api.LapsCtx(inputs.tiny_cfg(1), max_positions=64)
    g = torch.Generator(device="cuda").manual_seed(m + n + k)
    a, w = (torch.randint(-1, 2, (r, k), generator=g, device="cuda", dtype=torch.int8).to(torch.bfloat16) for r in (m, n))
    want = sum(a[:, c:c + (1 << 19)].float() @ w[:, c:c + (1 << 19)].float().T for c in range(0, k, 1 << 19))
    resid = torch.randint(-9, 10, (m, n), generator=g, device="cuda").float()
    assert torch.equal(ctx.laps_gemm_bf16(a, w), want)
    assert torch.equal(ctx.laps_gemm_epilogue_bf16(a, w, 1, resid=resid), resid + want)
    if n % 128 == 0:
        gate, up = want.double().view(m, n // 64, 2, 32).unbind(2)
        ref = (torch.nn.functional.silu(gate) * up).reshape(m, n // 2)
        got = ctx.laps_gemm_epilogue_bf16(a, w, 2).double()
        # the sums are exact; one bf16 rounding (at most 2^-8) and an fp32 SiLU, whose exponential of x is formed from a
        # product rounded to 2^-24 of |x|
        slack = 2.0 ** -8 + 2.0 ** -20 + (2.0 ** -22 * gate.abs()).reshape(m, n // 2)
        assert bool(((got - ref).abs() <= ref.abs() * slack + 1e-6).all())
    ctx.close()
