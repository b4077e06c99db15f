"""The attention whose workgroups take equal shares of the batch: shares that end inside a block of query rows, blocks cut
into many parts, several whole blocks per share, a workgroup for every block, sequences of no and of one token, rows of
padding, page-table entries that are unset or outside the pools, un-captured and in a captured graph, against float64.

Launches of 256-row blocks whose page tables are at least 80 pages wide (20 key tiles) take equal shares."""
import math

import numpy as np
import pytest
import torch

from gpu_harness import MAX_ABS_TOL, REL_L2_TOL, Case, errors
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


TURNS = [64, 1, 33, 64, 50, 0, 61, 40, 64, 64, 57, 48, 64, 64, 63, 64, 64, 64, 64, 64, 64]
TURNS_PRE = [4000, 0, 17, 2500, 700, 30, 64, 63, 1, 4096, 3333, 128, 129, 0, 512, 1024, 900, 77, 5, 4095, 2048]
CASES = {   # model, new tokens, cached tokens, least pages of the table, rows of padding behind every sequence, holes in it
    "one_long_chunk": (inputs.qwen32b_cfg, [2048], [0], 0, 0, False),        # 41 x 8 blocks of 1..32 tiles, 256 shares
    "ragged_chunk_over_prefix": (inputs.qwen32b_cfg, [1847], [6144], 0, 0, False),   # nearly every block is cut
    "many_turns": (inputs.qwen32b_cfg, TURNS, TURNS_PRE, 0, 0, False),
    "padded_turns": (inputs.qwen32b_cfg, TURNS, TURNS_PRE, 0, 9, False),
    "turns_with_unset_and_wild_pages": (inputs.qwen32b_cfg, TURNS, TURNS_PRE, 0, 0, True),
    "group_of_7": (inputs.qwen7b_cfg, [900, 300, 400], [0, 1500, 3000], 0, 0, False),    # 28 query heads over 4 kv heads
    "head_dim_64": (inputs.tiny_cfg, [4000, 3000, 64 * 9], [0, 100, 2000], 0, 0, False),
    "few_tiles": (inputs.tiny_cfg, [140] * 70 + [600], [0] * 70 + [50], 80, 0, False),   # whole blocks only, several a share
    "a_workgroup_per_block": (inputs.qwen32b_cfg, [40] * 15 + [64], [0] * 15 + [700], 80, 0, False),
    "few_blocks_padded": (inputs.qwen14b_cfg, [64, 0, 1, 52] * 4, [300, 0, 0, 17] * 4, 128, 3, False),
    "one_chunk_on_the_grid": (inputs.qwen32b_cfg, [1500], [2048], 0, 0, False),  # 240 blocks, not worth cutting
    "narrow_table": (inputs.qwen32b_cfg, [64] * 24, [1200] * 23 + [0], 79, 0, False),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_attention_in_equal_shares_matches_float64(name):
    cfgf, new, pre, width, pad, holes = CASES[name]
    cfg = cfgf(1)
    ctx = api.LapsCtx(cfg, 64)
    g = torch.Generator(device="cuda").manual_seed(len(name))
    cu = np.concatenate([[0], np.cumsum(np.asarray(new) + pad)])
    table, n_pages = inputs.make_page_table(11, new, pre)
    table = np.pad(table, ((0, 0), (0, max(0, width - table.shape[1]))), constant_values=-1)
    if holes:   # read as page 0
        for i, at in ((0, 3), (0, 200), (9, 0), (20, 77)):
            table[i, at] = -1
        table[3, 100], table[10, 5] = n_pages, 1 << 30
    draw = lambda shape, std=1.0: torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0, std, generator=g)
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.int32)).cuda()
    # scores spread wide enough (std about 2.5) for the running maximum to move between the parts of a block
    q = draw((int(cu[-1]), cfg.q_dim), 2.5)
    kp, vp = draw((n_pages, cfg.n_kv_heads, 16, cfg.head_dim)), draw((n_pages, cfg.n_kv_heads, cfg.head_dim, 16))
    lens = d(new) if pad else None
    got = ctx.laps_attention(d(cu), lens, d(pre), d(table), kp, vp, q).double().view(-1, cfg.n_q_heads, cfg.head_dim)
    again = ctx.laps_attention(d(cu), lens, d(pre), d(table), kp, vp, q).double().view(-1, cfg.n_q_heads, cfg.head_dim)
    for i, (n, h) in enumerate(zip(new, pre)):
        if n == 0:
            continue
        rows = slice(int(cu[i]), int(cu[i]) + n)
        assert torch.equal(got[rows], again[rows])
        ids = table[i, :(n + h + 15) // 16]
        pages = d(np.where((ids < 0) | (ids >= n_pages), 0, ids)).long()
        k = kp[pages].transpose(1, 2).reshape(-1, cfg.n_kv_heads, cfg.head_dim)[:n + h].double()
        v = vp[pages].permute(0, 3, 1, 2).reshape(-1, cfg.n_kv_heads, cfg.head_dim)[:n + h].double()
        want = reference(cfg, q[rows].double().view(n, cfg.n_q_heads, cfg.head_dim), k, v, h)
        err = (got[rows] - want).flatten(1).norm(dim=1)
        # probabilities and result are bf16 (2^-9 relative each, rms 1.7e-3 together); a token's heads share one norm
        assert bool((err <= 8e-3 * want.flatten(1).norm(dim=1)).all()), (name, i, float((err / want.flatten(1).norm(dim=1)).max()))
    ctx.close()


# bucket 64, depth 32, 4 query heads per kv head: 256-row blocks, a table of 90 pages
GRAPH_CFG = inputs.ModelCfg(512, 16, 4, 64, 512, 1)
FILLS = {
    "long_prefixes": ([64] * 20 + [1, 17, 64, 33], [1300, 0, 700] * 8),                  # cut
    "three_requests": ([64, 5, 40], [1200, 3, 0]),                                       # a workgroup per block
    "full_without_prefix": ([64] * 32, [0] * 32),                                        # whole blocks, none long
}


@pytest.mark.parametrize("name", sorted(FILLS))
def test_captured_graph_in_equal_shares_matches_the_oracle(name):
    new, pre = FILLS[name]
    case = Case(GRAPH_CFG, new, pre, 77)
    ctx = api.LapsCtx(GRAPH_CFG, max_positions=1440)
    case.to_device(ctx)
    table = np.pad(case.page_table, ((0, 0), (0, 90 - case.page_table.shape[1])), constant_values=-1)
    stream, d = torch.cuda.Stream(), lambda a: torch.from_numpy(np.ascontiguousarray(a, np.int32)).cuda()
    graph = ctx.laps_graph_capture(case.dev_layers, 64, 32, 90, case.k_pools, case.v_pools, stream)
    want, ks, vs, _ = case.oracle()
    d_new, d_pre, d_table, one = d(case.new_len), d(case.prefix_len), d(table), d([1])
    first = None
    for _ in range(3):
        # another fill and eager work in between: nothing may be left of either
        graph.laps_graph_stage(1, one, d([0]), d(table[:1]), case.d_x[:1].contiguous(), stream)
        out = torch.full((case.T, GRAPH_CFG.hidden), float("nan"), device="cuda")
        torch.cuda.synchronize()
        graph.laps_graph_stage(case.n, d_new, d_pre, d_table, case.d_x, stream)
        graph.laps_graph_replay(stream)
        graph.laps_graph_read_output(case.T, out, stream)
        torch.cuda.synchronize()
        rel, mx = errors(out.cpu().numpy(), want)
        assert rel < REL_L2_TOL and mx < MAX_ABS_TOL, (rel, mx)
        first = out if first is None else first
        assert torch.equal(out, first)
    k, v = case.gathered_new_kv(0)
    assert errors(k, np.concatenate(ks[0]))[0] < 4e-3 and errors(v, np.concatenate(vs[0]))[0] < 4e-3
    graph.close()
    ctx.close()
