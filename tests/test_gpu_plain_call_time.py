"""Timed calls in plain mode: the events around a call cost the host about as much
as its launch, not several times that.  Calls of 1,000 draws in a row with
per-call timing on take less than twice the time of those with it off (each the
best of several runs in turn)."""

import time

import pytest

pytestmark = pytest.mark.gpu


def test_timing_costs_less_than_the_call():
    import torch
    import paper_1411_2484_amd as ph
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    ctx = ph.Context(0, max_instances=1)
    ids = ctx.seed_instances(32, 913, 1, (9, 17), 0, 0)
    r = torch.empty(1000, dtype=torch.float64, device="cuda")
    reqs = ph.make_requests(ids, [1000], [0])
    best = {True: 1e9, False: 1e9}
    for _ in range(9):
        for on in best:
            ctx.set_timing(on)
            for call in range(1200):
                if call == 200:
                    torch.cuda.synchronize()
                    t = time.perf_counter()
                ctx.generate(reqs, None, None, r, mode=ph.PHPRNG_MODE_PLAIN)
            torch.cuda.synchronize()
            best[on] = min(best[on], time.perf_counter() - t)
    ctx.close()
    assert best[True] < 2 * best[False], "1,000 calls: %.1f ms timed, %.1f ms untimed" % (best[True] * 1e3,
                                                                                          best[False] * 1e3)
