"""The attention of page tables a few key tiles wide (64 keys, 4 pages each): 128-row blocks up to 2 tiles, up to 4 where they
spare a quarter of the rows or are more than two a compute unit, and up to 7 for launches of a block per compute unit at most;
256-row blocks else.  From 8 tiles on, few blocks are split over the keys: one tile per workgroup where all of them fit one
round of the 256 compute units and have at most 6400 rows of partial results, else four at least.  The rules on the host, both
sides of each of their edges against float64, and the same bits from 128- and 256-row blocks."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2601_11589_amd import api, inputs
from test_gpu_attention_shares import reference

# (model, new tokens, cached tokens, pages of the table, (query rows per workgroup, splits of the keys, least tiles of a split))
EDGES = [
    (inputs.qwen32b_cfg, [64] * 40, [0, 192, 17, 130] * 10, 16, (128, 1, 4)),       # 4 tiles, 1120 blocks, 320 rows a sequence
    (inputs.qwen32b_cfg, [64] * 40, [0, 192, 17, 193] * 10, 17, (256, 1, 4)),       # 5 tiles, as many blocks
    (inputs.qwen32b_cfg, [76] * 15, [0, 180, 17, 130, 52] * 3, 16, (128, 1, 4)),    # 472 blocks, 380 rows a sequence
    (inputs.qwen32b_cfg, [77] * 15, [0, 179, 17, 130, 51] * 3, 16, (256, 1, 4)),    # 385
    (inputs.qwen7b_cfg, [64] * 28, [0, 192, 136, 5] * 7, 16, (256, 1, 4)),          # 4 tiles, 504 blocks, 448 rows a sequence
    (inputs.qwen7b_cfg, [64] * 29, [0, 192, 136, 5] * 7 + [70], 16, (128, 1, 4)),   # 520 blocks
    (inputs.qwen32b_cfg, [64] * 8, [384, 0, 1, 200] * 2, 28, (128, 1, 4)),          # 7 tiles, 224 blocks
    (inputs.qwen32b_cfg, [64] * 8, [385, 0, 1, 200] * 2, 29, (128, 2, 4)),          # 8 tiles
    (inputs.qwen32b_cfg, [64] * 16, [384, 0, 1, 200] * 4, 28, (256, 1, 4)),         # 7 tiles, 448 blocks
    (inputs.qwen32b_cfg, [64] * 16, [385, 0, 1, 200] * 4, 29, (256, 1, 4)),         # 8 tiles
    (inputs.qwen32b_cfg, [1] * 4 + [63, 64] * 4, [0, 15] * 2 + [3, 384] * 4, 28, (128, 1, 4)),
    (inputs.qwen7b_cfg, [256, 129, 1, 77], [0, 127, 255, 64], 16, (128, 1, 4)),     # blocks of 18 tokens, the last of few rows
    (inputs.tiny_cfg, [65] * 120, [0, 63, 62, 31, 1] * 24, 8, (128, 1, 4)),         # head dimension 64, 2 tiles, 482 blocks
    (inputs.tiny_cfg, [65] * 120, [0, 63, 64, 31, 1] * 24, 9, (256, 1, 4)),         # 3 tiles
    (inputs.tiny_cfg, [65] * 60, [383] * 59 + [0], 28, (128, 1, 4)),                # 242 blocks of head dimension 64
    (inputs.tiny_cfg, [65] * 68, [383] * 67 + [0], 28, (256, 1, 4)),                # 274
    (inputs.qwen14b_cfg, [7], [900], 57, (128, 15, 1)),
    (inputs.qwen32b_cfg, [8], [2040], 128, (128, 32, 1)),                   # 8 blocks x 32 tiles
    (inputs.qwen32b_cfg, [8], [2041], 129, (128, 8, 4)),                    # 8 x 33
    (inputs.qwen7b_cfg, [9], [4087], 256, (128, 64, 1)),                    # 4 x 64, as many splits as there may be
    (inputs.qwen7b_cfg, [16], [3000], 189, (128, 48, 1)),                   # 112 rows x 48
    (inputs.qwen7b_cfg, [16], [4080], 256, (128, 16, 4)),                   # 112 x 64
    (inputs.qwen32b_cfg, [3, 5], [600, 0], 38, (128, 10, 1)),               # the second sequence is one split's
    (inputs.tiny_cfg, [100], [1900], 125, (128, 32, 1)),                    # rows that see no key of the last splits
    (inputs.tiny_cfg, [200, 64, 1], [321, 448, 511], 33, (128, 9, 1)),
]


def blocking(cfg, new, pages):
    out = (C.c_int64 * 6)()
    assert api.lib().laps_attn_plan_info(len(new), sum(new), cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, pages, out) == 0
    return out[0], out[2], out[3]


@pytest.mark.parametrize("case", range(len(EDGES)))
def test_blocks_of_a_few_key_tiles(case):
    cfgf, new, pre, pages, want = EDGES[case]
    assert max(-(-(n + h) // 16) for n, h in zip(new, pre)) <= pages
    assert blocking(cfgf(1), new, pages) == want


def operands(case, seed, pages):
    cfgf, new, pre, _, _ = EDGES[case]
    cfg = cfgf(1)
    g = torch.Generator(device="cuda").manual_seed(seed + case)
    cu = np.concatenate([[0], np.cumsum(new)])
    table, n_pages = inputs.make_page_table(5, new, pre)
    table = np.pad(table, ((0, 0), (0, pages - table.shape[1])), constant_values=-1)
    draw = lambda shape, std=1.0: torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0, std, generator=g)
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.int32)).cuda()
    q = draw((int(cu[-1]), cfg.q_dim), 2.5)
    kp, vp = draw((n_pages, cfg.n_kv_heads, 16, cfg.head_dim)), draw((n_pages, cfg.n_kv_heads, cfg.head_dim, 16))
    return cfg, new, pre, cu, d, table, kp, vp, q


@pytest.mark.gpu
@pytest.mark.parametrize("case,pages", [(0, 17), (2, 17), (5, 17), (12, 9)])
def test_blocks_of_128_and_256_rows_give_the_same_bits(case, pages):
    """A page table a page wider takes the launch to the other kind of block."""
    cfgf, new, _, narrow, _ = EDGES[case]
    assert blocking(cfgf(1), new, narrow)[0] == 128 and blocking(cfgf(1), new, pages)[0] == 256
    out = []
    for p in (narrow, pages):
        cfg, new, pre, cu, d, table, kp, vp, q = operands(case, 77, p)
        ctx = api.LapsCtx(cfg, 64)
        out.append(ctx.laps_attention(d(cu), None, d(pre), d(table), kp, vp, q))
        torch.cuda.synchronize()
        ctx.close()
    assert torch.equal(*out)


@pytest.mark.gpu
@pytest.mark.parametrize("case", range(len(EDGES)))
def test_attention_of_a_few_key_tiles_matches_float64(case):
    cfg, new, pre, cu, d, table, kp, vp, q = operands(case, 31, EDGES[case][3])
    ctx = api.LapsCtx(cfg, 64)
    run = lambda: ctx.laps_attention(d(cu), None, d(pre), d(table), kp, vp, q).double().view(-1, cfg.n_q_heads, cfg.head_dim)
    got = run()
    assert torch.equal(got, run())
    for i, (n, h) in enumerate(zip(new, pre)):
        rows = slice(int(cu[i]), int(cu[i]) + n)
        ids = d(table[i, :(n + h + 15) // 16]).long()
        k = kp[ids].transpose(1, 2).reshape(-1, cfg.n_kv_heads, cfg.head_dim)[:n + h].double()
        v = vp[ids].permute(0, 3, 1, 2).reshape(-1, cfg.n_kv_heads, cfg.head_dim)[:n + h].double()
        want = reference(cfg, q[rows].double().view(n, cfg.n_q_heads, cfg.head_dim), k, v, h)
        err = (got[rows] - want).flatten(1).norm(dim=1)
        # probabilities and result are bf16 (2^-9 relative each, rms 1.7e-3 together); a token's heads share one norm
        assert bool((err <= 8e-3 * want.flatten(1).norm(dim=1)).all()), (i, float((err / want.flatten(1).norm(dim=1)).max()))
    ctx.close()
