"""The launch that begins an un-captured batch (clamped lengths, attention work items, token positions, first RMSNorm):
more sequences than it scans in one pass, with rows of padding between them that hold NaN, lengths below 0 and above a
sequence's rows, and rows of one and of several loads per thread; against the oracle."""
import numpy as np
import pytest
import torch

from gpu_harness import MAX_ABS_TOL, REL_L2_TOL, Case, errors
from paper_2601_11589_amd import api, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden", [256, 1152])
def test_many_sequences_between_rows_of_padding(hidden):
    cfg = inputs.ModelCfg(hidden, 4, 2, 64, 512, 1)
    cap, given, used = 4, np.array([1, -2, 3, 9] * 75), np.array([1, 0, 3, 4] * 75)
    ids = np.flatnonzero(used)
    case = Case(cfg, used[ids], (ids * 7) % 50, 31)
    ctx = api.LapsCtx(cfg, max_positions=128)
    case.to_device(ctx)
    n = len(used)
    x = np.full((n * cap, hidden), np.nan, np.float32)
    prefix = np.zeros(n, np.int32)
    table = np.full((n, case.page_table.shape[1]), -1, np.int32)
    prefix[ids], table[ids] = case.prefix_len, case.page_table
    rows = np.concatenate([i * cap + np.arange(used[i]) for i in ids])
    x[rows] = case.x
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    y = ctx.laps_prefill_stack(case.dev_layers, d(np.arange(0, (n + 1) * cap, cap, dtype=np.int32)), d(given.astype(np.int32)),
                               d(prefix), d(table), case.k_pools, case.v_pools, d(x))
    torch.cuda.synchronize()
    got = y.cpu().numpy()[rows]
    want, ks, vs, _ = case.oracle()
    rel, mx = errors(got, want)
    assert np.isfinite(got).all() and rel < REL_L2_TOL and mx < MAX_ABS_TOL, (rel, mx)
    k, v = case.gathered_new_kv(0)
    assert errors(k, np.concatenate(ks[0]))[0] < 4e-3 and errors(v, np.concatenate(vs[0]))[0] < 4e-3
    ctx.close()
