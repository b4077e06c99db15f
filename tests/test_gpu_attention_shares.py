"""The attention whose workgroups take equal shares of the batch: shares that end inside a unit, units cut into many
parts, several whole units per share, sequences of no and of one token, against float64."""
import math

import numpy as np
import pytest
import torch

from paper_2601_11589_amd import api, inputs

pytestmark = pytest.mark.gpu


def reference(cfg, q, k, v, h):
    """Causal grouped-query attention of one sequence in float64; q [L, heads, hd], k / v [h + L, kv heads, hd]."""
    g = cfg.n_q_heads // cfg.n_kv_heads
    hidden = torch.arange(k.shape[0], device="cuda")[None] > torch.arange(q.shape[0], device="cuda")[:, None] + h
    out = torch.empty_like(q)
    for i in range(cfg.n_q_heads):
        s = (q[:, i] @ k[:, i // g].T) / math.sqrt(cfg.head_dim)
        out[:, i] = torch.softmax(s.masked_fill(hidden, -math.inf), -1) @ v[:, i // g]
    return out


CASES = {
    "one_long_chunk": (inputs.qwen32b_cfg, [2048], [0]),                     # 41 x 8 units of 1..32 tiles, 256 shares
    "ragged_chunk_over_prefix": (inputs.qwen32b_cfg, [1847], [6144]),        # nearly every unit is cut
    "many_turns": (inputs.qwen32b_cfg, [64, 1, 33, 64, 50, 0, 61, 40, 64, 64, 57, 48, 64, 64, 63, 64, 64, 64, 64, 64, 64],
                   [4000, 0, 17, 2500, 700, 30, 64, 63, 1, 4096, 3333, 128, 129, 0, 512, 1024, 900, 77, 5, 4095, 2048]),
    "group_of_7": (inputs.qwen7b_cfg, [900, 300, 400], [0, 1500, 3000]),     # 28 query heads over 4 kv heads
    "head_dim_64": (inputs.tiny_cfg, [4000, 3000, 64 * 9], [0, 100, 2000]),
    "few_tiles": (inputs.tiny_cfg, [140] * 70 + [600], [0] * 70 + [50]),     # fewer shares than workgroups
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_attention_in_equal_shares_matches_float64(name):
    cfgf, new, pre = CASES[name]
    cfg = cfgf(1)
    ctx = api.LapsCtx(cfg, 64)
    g = torch.Generator(device="cuda").manual_seed(len(name))
    cu = np.concatenate([[0], np.cumsum(new)])
    table, n_pages = inputs.make_page_table(11, new, pre)
    draw = lambda shape, std=1.0: torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0, std, generator=g)
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.int32)).cuda()
    # scores spread wide enough (std about 2.5) for the running maximum to move between the parts of a unit
    q = draw((int(cu[-1]), cfg.q_dim), 2.5)
    kp, vp = draw((n_pages, cfg.n_kv_heads, 16, cfg.head_dim)), draw((n_pages, cfg.n_kv_heads, cfg.head_dim, 16))
    got = ctx.laps_attention(d(cu), None, d(pre), d(table), kp, vp, q).double().view(-1, cfg.n_q_heads, cfg.head_dim)
    again = ctx.laps_attention(d(cu), None, d(pre), d(table), kp, vp, q).double().view(-1, cfg.n_q_heads, cfg.head_dim)
    assert torch.equal(got, again)
    for i, (n, h) in enumerate(zip(new, pre)):
        if n == 0:
            continue
        pages = d(table[i, :(n + h + 15) // 16]).long()
        k = kp[pages].transpose(1, 2).reshape(-1, cfg.n_kv_heads, cfg.head_dim)[:n + h].double()
        v = vp[pages].permute(0, 3, 1, 2).reshape(-1, cfg.n_kv_heads, cfg.head_dim)[:n + h].double()
        want = reference(cfg, q[cu[i]:cu[i + 1]].double().view(n, cfg.n_q_heads, cfg.head_dim), k, v, h)
        err = (got[cu[i]:cu[i + 1]] - want).flatten(1).norm(dim=1)
        # probabilities and result are bf16 (2^-9 relative each, rms 1.7e-3 together); a token's heads share one norm
        assert bool((err <= 8e-3 * want.flatten(1).norm(dim=1)).all()), (name, i, float((err / want.flatten(1).norm(dim=1)).max()))
    ctx.close()
