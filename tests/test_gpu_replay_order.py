"""A prepared replay follows the replay before it, and waits for nothing else: not
for a call on another stream that has since taken the staging slot of that
replay."""

import time

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ph():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1411_2484_amd as ph
    ph.lib()
    return ph


def _sleep_cycles(seconds):
    """torch's spin kernel takes clock cycles: how many last `seconds`."""
    import torch
    torch.cuda._sleep(1000)
    torch.cuda.synchronize()
    t = time.perf_counter()
    torch.cuda._sleep(1000000)
    torch.cuda.synchronize()
    return int(seconds / (time.perf_counter() - t) * 1000000)


def test_replay_does_not_wait_for_other_streams(ph):
    import torch
    ctx = ph.Context(0, max_instances=8)
    ids = ctx.seed_instances(32, 911, 8, (9, 17), 0, 0)
    counts, offs = np.full(4, 1000), np.arange(4) * 1000
    mine, other = ph.make_requests(ids[:4], counts, offs), ph.make_requests(ids[4:], counts, offs)
    r, r2 = (torch.empty(4000, dtype=torch.float64, device="cuda") for _ in range(2))
    cycles = _sleep_cycles(0.3)
    busy = torch.cuda.Stream()
    streams = [torch.cuda.Stream() for _ in range(4)]
    torch.cuda.synchronize()

    def overlaps(stream):
        with torch.cuda.stream(busy):
            torch.cuda._sleep(cycles)
        with torch.cuda.stream(stream):
            r2.zero_()
        stream.synchronize()
        free = not busy.query()
        torch.cuda.synchronize()
        return free

    free = [s for s in streams if overlaps(s)]
    if not free:
        pytest.skip("no stream of its own hardware queue")
    graph = ctx.graph(mine, None, None, r)
    graph.launch(free[0])
    torch.cuda.synchronize()
    for _ in range(7):  # the ring of eight staging slots comes round to the replay's
        ctx.generate(other, None, None, r2)
    torch.cuda.synchronize()
    with torch.cuda.stream(busy):
        torch.cuda._sleep(cycles)
        ctx.generate(other, None, None, r2, stream=busy)
    graph.launch(free[0])
    free[0].synchronize()
    assert not busy.query(), "the replay waited for a call on another stream"
    torch.cuda.synchronize()
    assert ctx.get_position(int(ids[0])) == 2000 and ctx.get_position(int(ids[4])) == 8000
    graph.close()
    ctx.close()
