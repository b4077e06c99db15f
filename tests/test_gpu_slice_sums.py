"""The row kernels behind a split K load the slices of a row in groups of up to eight before they add any: every number of
slices around those groups, rows of one to four pieces per workgroup, whole and ragged last pieces; the un-split product adds
the same numbers in another order."""
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
