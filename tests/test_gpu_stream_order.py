"""Work on a stream of the caller's own is ordered behind torch's current stream: by an event while that has work to run, by
nothing once it has run it all, and as before while either stream is being captured."""
import ctypes as C
import threading

import pytest
import torch

from paper_2601_11589_amd import api, inputs

pytestmark = pytest.mark.gpu


def idle(before, stream):
    return api.lib().laps_stream_idle(C.c_void_p(before.cuda_stream), C.c_void_p(stream.cuda_stream))


def busy(a, n=40):
    for _ in range(n):
        a = (a @ a).clamp_(-1, 1)
    return a


@pytest.mark.parametrize("own", [False, True])
def test_idle_is_reported_only_when_all_work_has_run(own):
    cur = torch.cuda.Stream() if own else torch.cuda.current_stream()
    other = torch.cuda.Stream()
    a = torch.ones((4096, 4096), dtype=torch.bfloat16, device="cuda")
    torch.cuda.synchronize()
    assert idle(cur, other) == 1
    with torch.cuda.stream(cur):
        busy(a)
        assert idle(cur, other) == 0          # some 10 ms of products are in flight
    cur.synchronize()
    assert idle(cur, other) == 1


@pytest.mark.parametrize("mode", ["global", "relaxed"])
def test_captures_are_neither_broken_nor_called_idle(mode):
    x, s = torch.zeros(64, device="cuda"), torch.cuda.Stream()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s, capture_error_mode=mode):
        x += 1
        assert idle(s, torch.cuda.Stream()) == 0 and idle(torch.cuda.default_stream(), s) == 0
        x += 1
    for _ in range(3):
        g.replay()
    torch.cuda.synchronize()
    assert float(x.sum()) == 6 * 64


@pytest.mark.parametrize("mode", ["global", "thread_local", "relaxed"])
@pytest.mark.parametrize("elsewhere", [False, True])
@pytest.mark.parametrize("own", [False, True])
def test_capture_of_a_third_stream_goes_on(mode, elsewhere, own):
    """A question about two streams that are not being captured leaves a capture of another one alone, asked by the thread
    that captures or by another one."""
    x, s, other = torch.zeros(64, device="cuda"), torch.cuda.Stream(), torch.cuda.Stream()
    before = torch.cuda.Stream() if own else torch.cuda.default_stream()
    torch.cuda.synchronize()
    g, said = torch.cuda.CUDAGraph(), []
    ask = lambda: said.append(idle(before, other))
    with torch.cuda.graph(g, stream=s, capture_error_mode=mode):
        x += 1
        if elsewhere:
            t = threading.Thread(target=ask)
            t.start()
            t.join()
        else:
            ask()
        x += 1
    assert said == [1]
    for _ in range(3):
        g.replay()
    torch.cuda.synchronize()
    assert float(x.sum()) == 6 * 64


def test_default_stream_is_busy_while_a_blocking_stream_is():
    """What is enqueued on the legacy default stream runs behind the work of every blocking stream, and so would an event."""
    handle = C.c_void_p()
    assert api.lib().hipStreamCreate(C.byref(handle)) == 0
    blocking, other = torch.cuda.ExternalStream(handle.value), torch.cuda.Stream()
    a = torch.ones((4096, 4096), dtype=torch.bfloat16, device="cuda")
    torch.cuda.synchronize()
    assert idle(torch.cuda.default_stream(), other) == 1
    with torch.cuda.stream(blocking):
        busy(a)
    assert idle(torch.cuda.default_stream(), other) == 0 and idle(blocking, other) == 0
    torch.cuda.synchronize()
    assert idle(torch.cuda.default_stream(), other) == 1 and idle(blocking, other) == 1
    assert api.lib().hipStreamDestroy(handle) == 0


def test_inputs_still_being_written_are_waited_for():
    ctx, stream = api.LapsCtx(inputs.tiny_cfg(1), 64), torch.cuda.Stream()
    g = torch.Generator(device="cuda").manual_seed(5)
    w = torch.randn((512, 256), device="cuda", generator=g).bfloat16()
    b = torch.randn((4096, 4096), device="cuda", generator=g).bfloat16()
    a = torch.zeros((300, 256), dtype=torch.bfloat16, device="cuda")
    value = torch.randn((300, 256), device="cuda", generator=g).bfloat16()
    want = ctx.laps_gemm_bf16(value, w)
    for _ in range(3):
        a.zero_()
        torch.cuda.synchronize()
        busy(b)
        a.copy_(value)
        got = ctx.laps_gemm_bf16(a, w, stream=stream)
        torch.cuda.synchronize()
        assert torch.equal(got, want)
    got = ctx.laps_gemm_bf16(a, w, stream=stream)   # nothing left to wait for
    torch.cuda.synchronize()
    assert torch.equal(got, want)
    ctx.close()
