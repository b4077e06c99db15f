"""A captured graph of many rows at different fills: the GEMMs choose their tile width and deal out their tiles by the
number of live rows they find on the device, so every fill has to give what the un-captured path gives, and what the
oracle gives for its first, middle and last sequence."""
import numpy as np
import pytest
import torch

from gpu_harness import MAX_ABS_TOL, REL_L2_TOL, errors, widen_layer
from oracle import laps_oracle
from paper_2601_11589_amd import api, inputs

pytestmark = pytest.mark.gpu

# q/k/v 3584 = 14 x 256 = 16 x 224 columns, o / down 2560 = 10 x 256 = 16 x 160: all three widths of either kind
CFG = inputs.ModelCfg(2560, 20, 4, 128, 1024, 1)
BUCKET, DEPTH = 64, 64


@pytest.fixture(scope="module")
def setup():
    ctx = api.LapsCtx(CFG, 256)
    layer = ctx.upload_layer(inputs.make_layer_weights(CFG, 5, 0))
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.empty((BUCKET * DEPTH, CFG.hidden), device="cuda").normal_(0, 1, generator=g)
    table = torch.arange(DEPTH * 4, dtype=torch.int32, device="cuda").view(DEPTH, 4)
    kp, vp = ctx.new_pools(DEPTH * 4, 1, zero=True)
    stream = torch.cuda.Stream()
    graph = ctx.laps_graph_capture([layer], BUCKET, DEPTH, 4, kp, vp, stream)
    yield ctx, layer, x, table, kp, vp, stream, graph
    graph.close()
    ctx.close()


@pytest.mark.parametrize("lens", [[1], [64] * 4, [64] * 4 + [1], [37] * 19 + [1], [64] * 31 + [63], [64] * 43 + [24],
                                  [64] * 64])
def test_every_fill_of_a_graph_matches_the_uncaptured_path(setup, lens):
    ctx, layer, x, table, kp, vp, stream, graph = setup
    n, rows = len(lens), sum(lens)
    d = lambda a: torch.from_numpy(np.asarray(a, np.int32)).cuda()
    live = torch.arange(BUCKET, device="cuda")[None] < torch.tensor(lens + [0] * (DEPTH - n), device="cuda")[:, None]   # [slot, token]

    def poison():                                     # nothing of another fill, or of the other path, may pass for written
        for pool in (kp[0], vp[0]):
            pool.fill_(776.0)
        torch.cuda.synchronize()

    def written():                                    # [token, kv head, head_dim] of K and V; every other slot untouched
        # pages 4 s .. 4 s + 3 hold slot s: K [page][head][16][hd], V [page][head][hd][16]
        k = kp[0].view(DEPTH, 4, CFG.n_kv_heads, 16, CFG.head_dim).transpose(2, 3).reshape(DEPTH, BUCKET, CFG.n_kv_heads, CFG.head_dim)
        v = vp[0].view(DEPTH, 4, CFG.n_kv_heads, CFG.head_dim, 16).permute(0, 1, 4, 2, 3).reshape(DEPTH, BUCKET, CFG.n_kv_heads, CFG.head_dim)
        assert bool((k[~live] == 776.0).all()) and bool((v[~live] == 776.0).all())
        assert not bool((k[live] == 776.0).all(-1).any()) and not bool((v[live] == 776.0).all(-1).any())
        return k[live].double(), v[live].double()

    poison()
    pre, out = d([0] * n), torch.empty((rows, CFG.hidden), device="cuda")
    graph.laps_graph_stage(n, d(lens), pre, table[:n].contiguous(), x[:rows].contiguous(), stream)
    graph.laps_graph_replay(stream)
    graph.laps_graph_read_output(rows, out, stream)
    torch.cuda.synchronize()
    k_graph, v_graph = written()
    cu, ids = np.concatenate([[0], np.cumsum(lens)]), sorted({0, n // 2, n - 1})
    picked = np.concatenate([np.arange(cu[i], cu[i + 1]) for i in ids])
    none = [[None] * len(ids)]
    exact, *_ = laps_oracle.stack_forward(CFG, [widen_layer(inputs.make_layer_weights(CFG, 5, 0))], x.cpu().numpy()[picked].astype(np.float64),
                                          [lens[i] for i in ids], none, none, False)
    rel, mx = errors(out.cpu().numpy()[picked], exact)
    assert rel < REL_L2_TOL and mx < MAX_ABS_TOL, (rel, mx)
    poison()
    want = ctx.laps_prefill_layer(layer, d(np.concatenate([[0], np.cumsum(lens)])), None, pre, table[:n].contiguous(), kp[0], vp[0],
                                  x[:rows].contiguous())
    torch.cuda.synchronize()
    # other K splits on the un-captured side: fp32 sums in another order, re-rounded to bf16 operands four times in the
    # layer (2^-9 / sqrt(3) each, in part of the elements)
    assert float((out - want).norm() / want.norm()) < 4 * 2.0 ** -9 / 3 ** 0.5
    k_want, v_want = written()
    assert float((k_graph - k_want).norm() / k_want.norm()) < 2.0 ** -9
    assert float((v_graph - v_want).norm() / v_want.norm()) < 2.0 ** -9
