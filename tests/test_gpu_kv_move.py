"""laps_kv_scatter / laps_kv_gather against plain indexing: sequences that begin and end in the middle of a page, of no
and of one token, unset table entries, and arrays that are not 16-byte aligned (bit-exact, all other slots untouched)."""
import numpy as np
import pytest
import torch

from paper_2601_11589_amd import api, inputs

pytestmark = pytest.mark.gpu


def aligned_or_not(shape, odd, g):
    n = int(np.prod(shape))
    flat = torch.empty(n + 8, dtype=torch.bfloat16, device="cuda").normal_(0, 1, generator=g)
    return flat[odd:odd + n].view(shape)


@pytest.mark.parametrize("odd", [0, 1])
@pytest.mark.parametrize("cfgf", [inputs.tiny_cfg, inputs.qwen7b_cfg])
@pytest.mark.parametrize("lens,start", [([1], [15]), ([16, 16], [0, 32]), ([17, 0, 3, 40, 1], [5, 9, 14, 31, 0]),
                                        ([0, 33, 100, 7], [3, 1, 16, 2000])])
def test_kv_scatter_and_gather_match_indexing(lens, start, cfgf, odd):
    cfg = cfgf(1)
    ctx = api.LapsCtx(cfg, 64)
    n, rows = len(lens), sum(lens)
    g = torch.Generator(device="cuda").manual_seed(rows * 7 + odd)
    table, n_pages = inputs.make_page_table(3, np.asarray(lens) + 1, np.asarray(start))
    table[n - 1, start[n - 1] // 16] = -1                      # unset entry: these tokens are not moved
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    d = lambda a: torch.from_numpy(np.asarray(a, np.int32)).cuda()
    k, v = (aligned_or_not((rows, cfg.n_kv_heads, cfg.head_dim), odd, g) for _ in range(2))
    kp = aligned_or_not((n_pages, cfg.n_kv_heads, 16, cfg.head_dim), odd, g)
    vp = aligned_or_not((n_pages, cfg.n_kv_heads, cfg.head_dim, 16), odd, g)
    want_k, want_v = kp.clone(), vp.clone()
    pages = np.full(rows, -1)
    for i in range(n):
        for t in range(lens[i]):
            pages[cu[i] + t] = table[i, (start[i] + t) // 16]
            if pages[cu[i] + t] >= 0:
                want_k[pages[cu[i] + t], :, (start[i] + t) % 16] = k[cu[i] + t]
                want_v[pages[cu[i] + t], :, :, (start[i] + t) % 16] = v[cu[i] + t]
    ctx.laps_kv_scatter(d(cu), d(start), d(table), k, v, kp, vp)
    assert torch.equal(kp.view(torch.int16), want_k.view(torch.int16))
    assert torch.equal(vp.view(torch.int16), want_v.view(torch.int16))
    got_k, got_v = ctx.laps_kv_gather(d(cu), d(start), d(table), kp, vp, rows)
    moved = torch.from_numpy(pages >= 0).cuda()
    assert torch.equal(got_k[moved], k[moved]) and torch.equal(got_v[moved], v[moved])
    ctx.close()
