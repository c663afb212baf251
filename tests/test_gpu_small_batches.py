"""Small batches: at most eight requests travel in the kernel arguments, more
are read from pinned or device memory; while SIMDs would idle, two or four
waves share a tile and divide its rows.  Request counts around eight, starts
and lengths around the edges of tiles and of their parts, through every entry
point in turn (generate, allocation-free, prepared replays on another stream),
bit for bit against the oracle.  Kernel times come from time stamps of the
kernels or, where those do not apply, from events; either lies between zero
and the time of the call on the host's clock (1% allowed for the two clocks)."""

import time

import numpy as np
import pytest

from tests.gpu_helpers import alloc_outputs, compare_request, to_host

pytestmark = pytest.mark.gpu

SEED = 0x14112484 + 6300


@pytest.fixture(scope="module")
def ph():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1411_2484_amd as ph
    ph.lib()
    return ph


def _heads_counts(k, tile):
    heads = [(0, 1, tile - 1, tile - 31, tile // 2 - 3, tile // 4 + 5, 3 * tile - 7)[i % 7] for i in range(k)]
    counts = [(1, 2 * tile + 3, tile // 4, tile // 2 + 1, 40, tile, tile + 33, 0, 5, 3 * tile // 4 - 1)[i * 7 % 10]
              for i in range(k)]
    return np.array(heads, dtype=np.uint64), np.array(counts, dtype=np.uint64)


@pytest.mark.parametrize("k", [1, 2, 8, 9, 70])
@pytest.mark.parametrize("width,sched", [(32, "skip"), (32, "constant"), (64, "skip"), (64, "constant"),
                                         (64, "restored")])
def test_requests_around_the_inline_limit(ph, orc, tab32, tab64, width, sched, k):
    import torch
    heads, counts = _heads_counts(k, 2048 if width == 32 or sched == "constant" else 1024)
    if k < 3:
        counts[0] = 1234
    offs = np.concatenate([[0], np.cumsum(counts)[:-1]]).astype(np.uint64) + np.uint64(3)
    n, e, _ = orc.seed(width, SEED + width, k, (9, 17, 3))
    p, a = orc.lcg_params(width)
    ctx = ph.Context(0, max_instances=k)
    s0 = np.arange(3, k + 3, dtype=np.uint64) * np.uint64(0x1234567890abc)
    if sched == "constant":
        ids = ctx.add_instances_skip(width, n, e, np.arange(1, k + 1, dtype=np.uint64), k0=heads)
        state = [(int(heads[i]) * (i + 1) % int(n[i]), 0) for i in range(k)]
    elif sched == "restored":
        ids = ctx.add_instances(width, n, e, s0=s0)
        state = [(0, int(s0[i])) for i in range(k)]
    else:
        ids = ctx.add_instances(width, n, e, k0=heads)
        tab = tab32 if width == 32 else tab64
        state = [orc.position(tab, p, a, int(n[i]), 0, 1, int(heads[i])) for i in range(k)]
    reqs = ph.make_requests(ids, counts, offs)
    side = torch.cuda.Stream()
    out = alloc_outputs(int(counts.sum()) + 6, width == 32, width == 64, True)
    graph = ctx.graph(reqs, *out)
    for call in ("generate", "noalloc", "replay", "replay", "R only"):
        torch.cuda.synchronize()
        if call == "replay":
            graph.launch(side)
        elif call == "noalloc":
            ctx.generate_noalloc(reqs, *out)
        else:
            ctx.generate(reqs, *(out if call == "generate" else (None, None, out[2])))
        torch.cuda.synchronize()
        hc32, hc64, hr = to_host(*out)
        got_c = None if call == "R only" else hc32 if width == 32 else hc64
        for i in range(k):
            cnt = int(counts[i])
            m, s = state[i]
            if sched == "constant":
                wc, wr, m = orc.generate_cskip(int(n[i]), int(e[i]), i + 1, m, cnt)
            else:
                wc, wr, m, s = orc.generate(p, a, int(n[i]), int(e[i]), m, s, cnt)
            state[i] = (m, s)
            if cnt:
                compare_request(got_c, hr, int(offs[i]), cnt, wc, wr, "%s, request %d" % (call, i))
    graph.close()
    ctx.close()


@pytest.mark.parametrize("shape", ["persistent", "plain", "no draws", "more waves than stamps", "width 64", "replay"])
def test_kernel_times(ph, shape):
    import torch
    width = 64 if shape == "width 64" else 32
    count = 0 if shape == "no draws" else 1 << 20
    ctx = ph.Context(0, max_instances=4)
    ids = ctx.seed_instances(width, 77, 4, (9, 17), 0, 0)
    r = torch.empty(4 * max(count, 1), dtype=torch.float64, device="cuda")
    reqs = ph.make_requests(ids, np.full(4, count), np.arange(4) * count)
    if shape == "more waves than stamps":
        ctx.set_tuning(block_threads=512, blocks_per_cu=8, tiles_per_chunk=1, unroll=4)
        reqs = ph.make_requests(ids, np.full(4, 12 << 20), np.arange(4) * (12 << 20))
        r = torch.empty(48 << 20, dtype=torch.float64, device="cuda")
    graph = ctx.graph(reqs, None, None, r) if shape == "replay" else None
    torch.cuda.synchronize()
    ctx.timing_reset()
    total = 0.0
    for call in range(11):  # more calls than staging slots
        t = time.perf_counter()
        if graph:
            graph.launch()
        else:
            ctx.generate(reqs, None, None, r, mode=ph.PHPRNG_MODE_PLAIN if shape == "plain" else ph.PHPRNG_MODE_PERSISTENT)
        torch.cuda.synchronize()
        host_ms = (time.perf_counter() - t) * 1e3
        ms = ctx.last_kernel_ms()
        assert 0 <= ms <= 1.01 * host_ms and (ms > 0 or count == 0)
        total += ms
    total_ms, calls = ctx.timing_read()
    assert calls == 11 and abs(total_ms - total) <= 1e-9 * total + 1e-12
    ctx.set_timing(False)
    ctx.generate(reqs, None, None, r)
    torch.cuda.synchronize()
    assert ctx.timing_read()[1] == 11
    if graph:
        graph.close()
    ctx.close()


@pytest.mark.parametrize("k", [3, 20])
def test_allocation_free_calls_under_capture(ph, orc, k):
    import torch
    ctx = ph.Context(0, max_instances=k)
    n, e, _ = orc.seed(32, SEED + 5, k, (9, 17))
    ids = ctx.add_instances(32, n, e)
    counts = np.arange(1, k + 1, dtype=np.uint64) * np.uint64(700)
    offs = np.concatenate([[0], np.cumsum(counts)[:-1]]).astype(np.uint64)
    r = torch.empty(int(counts.sum()), dtype=torch.float64, device="cuda")
    want = np.concatenate([orc.generate(*orc.lcg_params(32), int(n[i]), int(e[i]), 0, 1, int(counts[i]))[1]
                           for i in range(k)])
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, capture_error_mode="relaxed"):
        ctx.generate_noalloc(ph.make_requests(ids, counts, offs), None, None, r, stream=torch.cuda.current_stream())
    for _ in range(3):
        r.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(r.cpu().numpy().view(np.uint64), want.view(np.uint64))
    del g
    ctx.close()
