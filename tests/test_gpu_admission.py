"""Launches whose workgroups wait for each other take turns where they do not
fit the device together; what else a caller has on the streams is left alone."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

HOLD_MS = 400


def _hold(torch, stream, ms):
    """Keep a stream busy: one wave that waits."""
    with torch.cuda.stream(stream):
        torch.cuda._sleep(int(ms * _hold.per_ms))


@pytest.fixture(scope="module")
def hold(ea_gpu):
    import torch
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda._sleep(1000)
    a.record()
    torch.cuda._sleep(1_000_000)
    b.record()
    b.synchronize()
    _hold.per_ms = 1_000_000 / a.elapsed_time(b)
    return lambda stream, ms=HOLD_MS: _hold(torch, stream, ms)


def test_later_work_on_a_callers_stream_is_not_waited_for(ea_gpu, hold):
    """A run of L = 128 fills the device with its launch; after it its caller
    queues something long.  A run on another stream waits for the launch alone."""
    import torch
    a = ea_gpu.Sim(128, 0.4, 0.8, seed=1)
    others = [ea_gpu.Sim(64, 0.4, 0.8, seed=2) for _ in range(6)]
    want = ea_gpu.Sim(64, 0.4, 0.8, seed=2)
    want.sweep(9)
    x = torch.zeros(1, device="cuda")
    torch.cuda.synchronize()
    tried = 0
    for b in others:
        # streams may share a hardware queue: take one that runs beside a's
        hold(a._stream)
        with torch.cuda.stream(b._stream):
            x.add_(1.0)
        b._stream.synchronize()
        beside = not a._stream.query()
        a._stream.synchronize()
        if not beside:
            continue
        tried += 1
        a.sweep(3)
        hold(a._stream)
        b.sweep(9)
        b.sync()
        assert not a._stream.query(), "the run waited for its neighbour's later work"
        a.sync()
        assert all(np.array_equal(b.spins(r), want.spins(r)) for r in (0, 1))
        break
    assert tried, "no two streams ran side by side"
    for s in [a, want] + others:
        s.close()


def test_a_listed_stream_can_be_captured(ea_gpu):
    """A caller captures on a stream that has had a launch, while another
    thread's run needs the whole device."""
    import torch
    a, b, want = (ea_gpu.Sim(128, 0.4, 0.8, seed=s) for s in (1, 2, 2))
    a.sweep(3)
    a.sync()
    want.sweep(4)
    x, y = torch.arange(1000, device="cuda"), torch.zeros(1000, dtype=torch.int64, device="cuda")
    torch.cuda.synchronize()

    def other():
        b.sweep(4)
        b.sync()

    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=a._stream, capture_error_mode="thread_local"):
        y.copy_(x * 2)
        t = threading.Thread(target=other)
        t.start()
        t.join()
    for k in range(3):
        y.zero_()
        x.add_(1)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, x * 2), k
    assert all(np.array_equal(b.spins(r), want.spins(r)) for r in (0, 1))
    a.sweep(2)
    a.sync()
    for s in (a, b, want):
        s.close()


@pytest.mark.parametrize("L", [16, 64, 128])
def test_a_captured_sweep_runs_at_its_replay(ea_gpu, L):
    """Captured by the caller, a sweep does nothing until the graph runs, and
    then what it does eagerly."""
    import torch
    a, want = (ea_gpu.Sim(L, 0.4, 0.8, seed=3) for _ in range(2))
    for s in (a, want):
        s.sweep(2)
        s.sync()
    before = [a.spins(r) for r in (0, 1)]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=a._stream, capture_error_mode="thread_local"):
        a.sweep(5)
    torch.cuda.synchronize()
    assert all(np.array_equal(a.spins(r), before[r]) for r in (0, 1))
    graph.replay()
    torch.cuda.synchronize()
    want.sweep(5)
    want.sync()
    assert all(np.array_equal(a.spins(r), want.spins(r)) for r in (0, 1))
    a.close()
    want.close()
