"""Kernel times of many accumulate calls read at once: more launches than the
battery keeps pending (1024), so that it folds the finished ones in between.
Every launch is counted, and their total lies between zero and the time of the
calls on the host's clock (1% allowed for the two clocks)."""

import time

import pytest

pytestmark = pytest.mark.gpu


def test_times_of_many_calls():
    import torch
    import paper_1411_2484_amd as ph
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    calls, blocks = 400, 4
    r = torch.rand(blocks << 20, dtype=torch.float64, device="cuda")
    bat = ph.Battery(0)
    bat.accumulate(r)
    torch.cuda.synchronize()
    bat.reset()
    torch.cuda.synchronize()
    t = time.perf_counter()
    for _ in range(calls):
        bat.accumulate(r)
    torch.cuda.synchronize()
    host_ms = (time.perf_counter() - t) * 1e3
    times = bat.timing()
    assert [n for _, n in times.values()] == [calls] * len(times)
    assert all(ms > 0 for ms, _ in times.values())
    assert sum(ms for ms, _ in times.values()) <= 1.01 * host_ms
    bat.close()
