"""The memory samples of the latency model are device times: the time to read cached K/V is that of the bytes, not that of
launching the copies, and the model's linear terms describe it."""
import pytest

from paper_2601_11589_amd import api, inputs, latency_fit

pytestmark = pytest.mark.gpu


def test_memory_samples_follow_the_bytes():
    cfg = inputs.ModelCfg(5120, 40, 8, 128, 6912, 4)     # the 32B attention and cache, a quarter of its MLP
    ctx = api.LapsCtx(cfg, 33000)
    layers = [ctx.upload_layer(inputs.make_layer_weights(cfg, 1, 0))] * 4
    samples = latency_fit.collect_samples(ctx, layers, [16, 2048], [0, 8192, 16384, 32768])
    read = {h: min(s["kv_read_us"] for s in samples if s["H"] == h) for h in (8192, 16384, 32768)}
    # 4 layers x 4 KB a token, read and written once each, at 2.5 TB/s (a third of the memory's) to 16 TB/s (twice it: a
    # layer's 33 to 134 MB are partly in the memory-side cache, and the launches that run beside the copies are
    # subtracted); at the host's pace of launching 4 x 30 us and more, 8192 tokens would be at 2.2
    for h, us in read.items():
        assert 2.0 * 4 * 4096 * h / 16e6 <= us <= 2.0 * 4 * 4096 * h / 2.5e6, read
    assert read[32768] > 2.5 * read[8192], read
    fit = latency_fit.fit_and_boundaries(samples, cfg, 4, report_hist=(0, 8192, 32768))
    assert fit["r2_mem"] > 0.9 and fit["gamma_r"] > 0, fit
    ctx.close()
