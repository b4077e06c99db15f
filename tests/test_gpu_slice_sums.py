"""The row kernels behind a split K load the slices of a row in groups of up to eight before they add any: every number of
slices around those groups, rows of one to four pieces per workgroup, whole and ragged last pieces; the un-split product adds
the same numbers in another order.  The kernels of q/k/v and of SwiGLU are called directly, with rows one by one and turned
over, padding among them."""
import ctypes as C
import math

import numpy as np
import pytest
import torch

from paper_2601_11589_amd import api, inputs

from gpu_harness import errors

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1280, 2048, 2176, 5120, 8192])      # pieces of 2048 columns
@pytest.mark.parametrize("splits", [(1, 2, 3, 4, 5), (6, 7, 8, 9), (12, 16, 17, 24)])
def test_slices_added_in_any_number(n, splits):
    rng = np.random.default_rng(n)
    ctx = api.LapsCtx(inputs.tiny_cfg(1), max_positions=4096)
    try:
        for split in splits:
            m, k = 1 + split % 3, 128 * split
            a, w = (inputs.f32_to_bf16_bits((rng.standard_normal(s) * f).astype(np.float32)) for s, f in (((m, k), 1.0), ((n, k), 0.05)))
            want = inputs.bf16_bits_to_f64(a) @ inputs.bf16_bits_to_f64(w).T
            got = ctx.laps_gemm_bf16(api.bf16_tensor(a), api.bf16_tensor(w), split_k=split)
            torch.cuda.synchronize()
            assert ctx.laps_gemm_plan_info(m, n, k, split)["split"] == split
            rel, mx = errors(got.cpu().numpy(), want)
            # fp32 accumulation of exact bf16 products, at most k + split roundings of 2^-24 of partial sums of about 0.05 sqrt(k)
            assert rel < 2e-6 and mx < 1e-4 * math.sqrt(k), (split, rel, mx)
    finally:
        ctx.close()


SPLITS = (1, 2, 3, 4, 5, 6, 7, 8, 9, 12, 16, 17)


@pytest.mark.parametrize("rows", [1, 37, 129, 200])      # up to 128 one by one, v turned over above
@pytest.mark.parametrize("n_q,n_kv,hd,bias", [(4, 2, 64, False), (10, 2, 128, True)])
def test_qkv_of_any_number_of_slices(rows, n_q, n_kv, hd, bias):
    g = torch.Generator(device="cuda").manual_seed(rows + hd)
    width, pages, max_pos = (n_q + 2 * n_kv) * hd, 40, 512
    rope = torch.rand((max_pos, hd // 2, 2), device="cuda", generator=g) * 2 - 1
    b = torch.randn(width, device="cuda", generator=g).bfloat16() if bias else None
    pos = torch.randint(0, max_pos, (rows,), device="cuda", generator=g).int()
    slot = torch.randperm(pages * 16, device="cuda", generator=g)[:rows].int()
    slot[16:32] = torch.arange(pages * 16, pages * 16 + 16, device="cuda").int()[:max(0, min(rows, 32) - 16)]      # side by side in a page
    pos[torch.rand(rows, device="cuda", generator=g) < 0.2] = -1
    pos[32:48] = -1                                                                                   # padding only
    live = pos >= 0
    p = lambda t: C.c_void_p(t.data_ptr() if t is not None else 0)
    for split in SPLITS:
        part = torch.randn((split, rows, width), device="cuda", generator=g)
        part[:, ~live] = float("nan")
        q = torch.full((rows, n_q, hd), 7.0, dtype=torch.bfloat16, device="cuda")
        k = torch.full((pages + 1, n_kv, 16, hd), 7.0, dtype=torch.bfloat16, device="cuda")
        v = torch.full((pages + 1, n_kv, hd, 16), 7.0, dtype=torch.bfloat16, device="cuda")
        assert api.lib()._Z19laps_launch_epi_qkvPKfiPKtPKiS4_PK15HIP_vector_typeIfLj2EEiPtS9_S9_iiiiP12ihipStream_t(
            p(part), C.c_int(split), p(b), p(pos), p(slot), p(rope), C.c_int(max_pos), p(q), p(k), p(v), C.c_int(rows), C.c_int(n_q),
            C.c_int(n_kv), C.c_int(hd), C.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
        torch.cuda.synchronize()
        x = part[:, live].double().sum(0) + (b.double() if bias else 0)
        x = x.view(-1, n_q + 2 * n_kv, hd)
        lo, hi = x[..., :hd // 2], x[..., hd // 2:]
        cs = rope[pos[live].long()].double()[:, None]
        turned = torch.cat([lo * cs[..., 0] - hi * cs[..., 1], hi * cs[..., 0] + lo * cs[..., 1]], -1)
        at, page, off = slot[live].long(), slot[live].long() // 16, slot[live].long() % 16
        # one bf16 rounding of fp32 sums of split + 3 terms of about 1, which err by at most (split + 3)^2 2^-24 or so
        close = lambda got, want: bool(((got.double() - want).abs() <= want.abs() * 2.0 ** -8 + 6e-5).all())
        assert close(q[live], turned[:, :n_q]) and bool((q[~live] == 0).all()), split
        assert close(k[page, :, off], turned[:, n_q:n_q + n_kv]) and close(v[page, :, :, off], x[:, n_q + n_kv:]), split
        used = torch.zeros((pages + 1) * 16, dtype=torch.bool, device="cuda")
        used[at] = True
        assert bool((k.transpose(1, 2).reshape(-1, n_kv, hd)[~used] == 7).all()) and bool((v.permute(0, 3, 1, 2).reshape(-1, n_kv, hd)[~used] == 7).all())


@pytest.mark.parametrize("rows,inter", [(1, 64), (5, 1088), (130, 512)])
def test_swiglu_of_any_number_of_slices(rows, inter):
    g = torch.Generator(device="cuda").manual_seed(rows + inter)
    live = torch.rand(rows, device="cuda", generator=g) < 0.8
    live[0] = True
    flags = torch.where(live, 3, -1).int()
    p = lambda t: C.c_void_p(t.data_ptr())
    for split in SPLITS:
        part = torch.randn((split, rows, 2 * inter), device="cuda", generator=g)
        act = torch.full((rows + 1, inter), 7.0, dtype=torch.bfloat16, device="cuda")
        assert api.lib()._Z22laps_launch_epi_swigluPKfiPtiiPKiP12ihipStream_t(
            p(part), C.c_int(split), p(act), C.c_int(rows), C.c_int(inter), p(flags), C.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
        gate, up = part[:, live].double().sum(0).view(-1, inter // 32, 2, 32).unbind(2)
        want = (torch.nn.functional.silu(gate) * up).reshape(-1, inter)
        # one bf16 rounding; the device's exp and fp32 sums err by some 2^-20 of operands up to 20
        assert bool(((act[:rows][live].double() - want).abs() <= want.abs() * 2.0 ** -8 + 4e-4).all()), split
        assert bool((act[:rows][~live] == 7).all()) and bool((act[rows] == 7).all())
