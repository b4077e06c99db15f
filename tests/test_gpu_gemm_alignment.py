"""Operands and results of the GEMMs that are aligned to their elements only, and to 4 and 8 bytes: products of their own on every
plan they can have (up to 64 and 128 rows, one and several row tiles, K split or not, 64-, 128- and 256-column tiles, SwiGLU of 192
columns, rows of 2^22 values), against float64 with guard values around the result; and a layer and a captured graph whose weights
lie two bytes off, against the same weights in place."""
import ctypes as C

import pytest
import torch

from paper_2601_11589_amd import api, inputs

PARTIAL, RESID, SWIGLU = 0, 1, 2


def off(t, by):
    """The same values `by` elements behind a 256-byte bound."""
    buf = torch.empty(t.numel() + 128, dtype=t.dtype, device="cuda")
    assert buf.data_ptr() % 256 == 0
    v = buf[by:by + t.numel()].view(t.shape)
    v.copy_(t)
    return v


def guarded(shape, dtype, by):
    n = shape[0] * shape[1]
    buf = torch.full((n + 128,), 7.0, dtype=dtype, device="cuda")
    return buf, buf[by:by + n].view(shape)


SHAPES = [(3, 384, 320, PARTIAL), (8, 192, 192, RESID), (40, 5120, 5120, PARTIAL), (64, 27648, 5120, SWIGLU), (100, 512, 13824, RESID),
          (128, 256, 1088, SWIGLU), (129, 192, 1088, SWIGLU), (129, 192, 576, PARTIAL), (300, 3584, 1024, RESID), (700, 5120, 1088, SWIGLU),
          (1537, 5120, 256, RESID), (600, 7168, 5120, PARTIAL), (4, 128, (1 << 22) + 64, PARTIAL)]


@pytest.mark.gpu
@pytest.mark.parametrize("a_off,w_off", [(1, 0), (0, 1), (2, 4), (0, 0)])      # elements of 2 bytes
@pytest.mark.parametrize("m,n,k,epi", SHAPES)
def test_product_of_operands_off_their_bounds_matches_float64(m, n, k, epi, a_off, w_off):
    print(m, n, k, epi, a_off, w_off, flush=True)
    ctx = api.LapsCtx(inputs.tiny_cfg(1), max_positions=64)
    g = torch.Generator(device="cuda").manual_seed(m + n + k)
    a = off(torch.empty((m, k), dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g), a_off)
    w = off(torch.empty((n, k), dtype=torch.bfloat16, device="cuda").normal_(0, 0.02, generator=g), w_off)
    c = 1 << 18
    want = sum(a[:, i:i + c].double() @ w[:, i:i + c].double().T for i in range(0, k, c))
    info = ctx.laps_gemm_plan_info(m, n, k, 0, epi)
    ws = torch.empty(max(256, info["split"] * m * n * 4), dtype=torch.uint8, device="cuda")
    p, i32, st = (lambda t: C.c_void_p(t.data_ptr())), C.c_int32, C.c_void_p(torch.cuda.current_stream().cuda_stream)
    if epi == SWIGLU:
        buf, out = guarded((m, n // 2), torch.bfloat16, 1)
        rc = api.lib().laps_gemm_epilogue_bf16(ctx._h, p(a), p(w), i32(m), i32(n), i32(k), i32(2), None, None, p(out), p(ws), C.c_size_t(ws.numel()), st)
        gate, up = want.view(m, n // 64, 2, 32).unbind(2)
        ref = (torch.nn.functional.silu(gate) * up).reshape(m, n // 2)
        # one bf16 rounding (at most 2^-8 of the value) of fp32 sums: k products, std 0.02 sqrt(k), in a random walk of k / 16
        # roundings of 2^-24; six standard deviations are delta, silu' is below 1.1
        delta = 6 * 2.0 ** -24 * 0.02 * k / 4
        slack = (delta * (1.1 * up.abs() + gate.abs())).reshape(m, n // 2) + 1e-6
        ok = bool(((out.double() - ref).abs() <= ref.abs() * 2.0 ** -8 + slack).all())
    elif epi == RESID:
        resid = off(torch.empty((m, n), device="cuda").normal_(0, 4, generator=g), 1)
        buf, out = guarded((m, n), torch.float32, 1)
        rc = api.lib().laps_gemm_epilogue_bf16(ctx._h, p(a), p(w), i32(m), i32(n), i32(k), i32(1), p(resid), p(out), None, p(ws), C.c_size_t(ws.numel()), st)
        ref = want + resid.double()
        ok = float((out.double() - ref).norm() / ref.norm()) < 2e-6          # fp32 sums of exact products
    else:
        buf, out = guarded((m, n), torch.float32, 1)
        rc = api.lib().laps_gemm_bf16(ctx._h, p(a), p(w), p(out), i32(m), i32(n), i32(k), i32(0), p(ws), C.c_size_t(ws.numel()), st)
        # an fp32 sum of k products takes up to k / 32 / slices roundings of 2^-24 one after the other
        ok = float((out.double() - want).norm() / want.norm()) < (2e-6 if k < 1 << 20 else 2e-5)
    assert rc == 0, api.lib().laps_last_error()
    assert ok
    assert bool((buf[:1] == 7).all()) and bool((buf[1 + out.numel():] == 7).all())
    ctx.close()


@pytest.mark.gpu
@pytest.mark.parametrize("graph", [False, True])
def test_layer_with_weights_off_their_bounds(graph):
    """The products of a layer and of a captured graph of more than 256 rows: the same results as with weights in place but for
    the order of fp32 sums (a sum that falls to the other side of a bf16 bound moves a value by 2^-8)."""
    cfg = inputs.tiny_cfg(1)
    ctx = api.LapsCtx(cfg, max_positions=512)
    g = torch.Generator(device="cuda").manual_seed(5)
    draw = lambda shape, std=1.0, mean=0.0, dtype=torch.bfloat16: torch.empty(shape, dtype=dtype, device="cuda").normal_(mean, std, generator=g)
    d, i = cfg.hidden, cfg.intermediate
    w = {"ln1": draw((d,), 0.02, 1.0), "w_qkv": draw((cfg.qkv_dim, d), 0.05), "w_o": draw((d, cfg.q_dim), 0.05), "ln2": draw((d,), 0.02, 1.0),
         "w_down": draw((d, i), 0.05), "w_gate_up": ctx.laps_pack_gate_up(draw((i, d), 0.05), draw((i, d), 0.05))}
    moved = {k: (off(t, 1) if k.startswith("w_") else t) for k, t in w.items()}
    new, pre = [64, 3, 50, 64, 64, 40, 64, 17], [0, 40, 7, 100, 0, 16, 33, 5]
    table, n_pages = inputs.make_page_table(5, new, pre)
    i32 = lambda v: torch.tensor(v, dtype=torch.int32, device="cuda")
    cu = [0]
    for n in new:
        cu.append(cu[-1] + n)
    pools = draw((n_pages, cfg.n_kv_heads, 16, cfg.head_dim)), draw((n_pages, cfg.n_kv_heads, cfg.head_dim, 16))
    x = draw((cu[-1], d), dtype=torch.float32)
    outs = []
    for weights in (w, moved):
        kp, vp = pools[0].clone(), pools[1].clone()
        out = torch.empty_like(x)
        t = torch.from_numpy(table).int().cuda()
        if graph:
            s = torch.cuda.Stream()
            gr = ctx.laps_graph_capture([weights], 64, 8, t.shape[1], [kp], [vp], s)
            gr.laps_graph_stage(8, i32(new), i32(pre), t, x, s)
            for _ in range(3):
                gr.laps_graph_replay(s)
            gr.laps_graph_read_output(cu[-1], out, s)
            s.synchronize()
        else:
            ctx.laps_prefill_layer(weights, i32(cu), None, i32(pre), t, kp, vp, x, out)
        torch.cuda.synchronize()
        outs.append((out.double(), kp.double(), vp.double()))
    for a, b in zip(*outs):
        assert float((a - b).norm() / a.norm()) < 2e-3
    ctx.close()
