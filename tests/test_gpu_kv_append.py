"""The append of k and v behind the q/k/v projection: above 128 rows v goes out 8 tokens at a time where these lie side by
side in an aligned half of a page and one by one where not, 16 rows of the batch per workgroup whatever sequences they
belong to; up to 128 rows one by one.
Layer 0's v does not depend on the position, so the same rows appended at other starts are the same bits."""
import numpy as np
import pytest
import torch

from gpu_harness import Case, errors
from paper_2601_11589_amd import api, inputs

pytestmark = pytest.mark.gpu

LENS = {104: [1, 7, 8, 9, 40, 16, 23], 128: [1, 7, 8, 9, 40, 16, 47], 129: [1, 7, 8, 9, 40, 16, 48], 229: [1, 7, 8, 9, 40, 64, 100]}


def appended(ctx, cfg, lens, start):
    case = Case(cfg, lens, start, 4242).to_device(ctx)
    case.run_stack()
    k, v = case.gathered_new_kv(0)
    left = [int((p.view(torch.int16) == 0x7FC0).sum()) for p in (case.k_pools[0], case.v_pools[0])]
    unwritten = (case.n_pages * 16 - case.T - int(np.sum(start))) * cfg.n_kv_heads * cfg.head_dim
    assert left == [unwritten, unwritten]                      # nothing but the batch's own slots was written
    return case, k, v


@pytest.mark.parametrize("rows", sorted(LENS))
@pytest.mark.parametrize("cfg", [inputs.tiny_cfg(1), inputs.ModelCfg(256, 6, 3, 128, 512, 1)])
def test_appended_v_does_not_depend_on_where_the_rows_start(cfg, rows):
    ctx = api.LapsCtx(cfg, max_positions=256)
    lens = LENS[rows]
    assert sum(lens) == rows
    case, k0, v0 = appended(ctx, cfg, lens, [0] * len(lens))
    _, ks, vs, _ = case.oracle()
    # one bf16 rounding of the normed row (2^-9 rms), one of the result: below 4e-3 relative
    assert errors(k0, np.concatenate(ks[0]))[0] < 4e-3 and errors(v0, np.concatenate(vs[0]))[0] < 4e-3
    for start in ([1] * 7, [7, 9, 8, 15, 3, 8, 1], [8] * 7, [15, 1, 24, 16, 40, 0, 7]):
        _, _, v = appended(ctx, cfg, lens, start)
        assert np.array_equal(v, v0), start
    ctx.close()
