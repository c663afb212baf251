"""A captured call carries its request list: replays repeat it whatever other
lists the context has planned since, through every entry point that a stream
capture accepts, with list lengths around the requests that fit the kernel
arguments and those that one launch writes.  Between the replays the same
entry points run other lists (fewer and more requests, longer and shorter ones,
the other width), so that a replay that read a staging block of its context
would find another list there.  Bit for bit against the oracle."""

import numpy as np
import pytest

from tests.gpu_helpers import compare_request

pytestmark = pytest.mark.gpu

SEED = 0x14112484 + 6500


@pytest.fixture(scope="module")
def ph():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1411_2484_amd as ph
    ph.lib()
    return ph


def _requests(ph, ids, counts):
    counts = np.asarray(counts, dtype=np.uint64)
    return ph.make_requests(ids, counts, np.concatenate([[0], np.cumsum(counts)[:-1]]).astype(np.uint64))


@pytest.mark.parametrize("k", [8, 9, 60, 61, 121, 1100])
@pytest.mark.parametrize("entry", ["noalloc", "generate", "plain", "prepared"])
def test_replays_repeat_the_captured_list(ph, orc, entry, k):
    import torch
    ctx = ph.Context(0, max_instances=k + 260)
    n, e, _ = orc.seed(32, SEED + k, k, (9, 17))
    ids = ctx.add_instances(32, n, e)
    counts = 1 + np.arange(k, dtype=np.uint64) * np.uint64(7919) % np.uint64(700 if k > 200 else 5000)
    reqs = _requests(ph, ids, counts)
    r = torch.empty(int(counts.sum()), dtype=torch.float64, device="cuda")
    # the lists of the calls in between, on instances of their own
    o32 = ctx.seed_instances(32, SEED + 1, 200, (9, 17), 0, 1 << 40)
    o64 = ctx.seed_instances(64, SEED + 2, 60, (9, 17), 0, 1 << 30)
    others = [_requests(ph, np.concatenate([o64, o32]), [6000] * 60 + [40] * 200),
              _requests(ph, o64[:12], [30000] * 12), _requests(ph, o32[:9], [1] * 9)]
    room = torch.empty(400000, dtype=torch.float64, device="cuda")
    prepared = ctx.graph(reqs, None, None, r) if entry == "prepared" else None
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, capture_error_mode="relaxed"):
        stream = torch.cuda.current_stream()
        if entry == "noalloc":
            ctx.generate_noalloc(reqs, None, None, r, stream=stream)
        elif entry == "prepared":
            prepared.launch(stream)
        else:
            ctx.generate(reqs, None, None, r, stream=stream,
                         mode=ph.PHPRNG_MODE_PLAIN if entry == "plain" else ph.PHPRNG_MODE_PERSISTENT)
    assert [ctx.get_position(int(ids[i])) for i in range(3)] == [int(c) for c in counts[:3]]
    p, a = orc.lcg_params(32)
    want = [orc.generate(p, a, int(n[i]), int(e[i]), 0, 1, int(counts[i]))[1] for i in range(k)]
    for replay in range(4):
        r.fill_(-1.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        got = r.cpu().numpy()
        for i in range(k):
            compare_request(None, got, int(reqs["out_offset"][i]), int(counts[i]), None, want[i],
                            "replay %d, request %d of %d" % (replay, i, k))
        other = others[replay % 3]
        ctx.generate_noalloc(other, None, None, room)
        for _ in range(9):  # more calls than staging slots
            ctx.generate(other, None, None, room)
        torch.cuda.synchronize()
    del graph
    if prepared:
        prepared.close()
    ctx.close()


@pytest.mark.parametrize("k", [3, 20])
def test_width64_replays_from_the_captured_states(ph, orc, k):
    """The device holds the messages of width-64 pseudorandom-skip instances:
    replays repeat their draws when the instances are set back before each."""
    import torch
    ctx = ph.Context(0, max_instances=2 * k)
    p, a = orc.lcg_params(64)
    n, e, _ = orc.seed(64, SEED + 3, 2 * k, (9, 17))
    s0 = np.where(np.arange(2 * k) % 2, np.uint64(1), np.arange(3, 2 * k + 3).astype(np.uint64) * np.uint64(0x1234567890abc))
    ids = ctx.add_instances(64, n, e, s0=s0)  # tile starts from the table, and from the carried state
    starts = [ctx.get_state(int(i)) for i in ids]
    counts = 100 + np.arange(2 * k) * 300
    reqs = _requests(ph, ids, counts)
    c, r = torch.empty(int(counts.sum()), dtype=torch.int64, device="cuda"), None
    want = [orc.generate(p, a, int(n[i]), int(e[i]), 0, int(s0[i]), int(counts[i]))[0] for i in range(2 * k)]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, capture_error_mode="relaxed"):
        ctx.generate_noalloc(reqs, None, c, r, stream=torch.cuda.current_stream())
    for replay in range(3):
        c.fill_(-1)
        if replay:
            for i, (m, s, _, pos) in zip(ids, starts):
                ctx.set_state(int(i), m, s, pos)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        got = c.cpu().numpy().view(np.uint64)
        for i in range(2 * k):
            compare_request(got, None, int(reqs["out_offset"][i]), int(counts[i]), want[i], None,
                            "replay %d, request %d" % (replay, i))
        ctx.generate(reqs, None, c, r)
    torch.cuda.synchronize()
    del graph
    ctx.close()


def test_replays_after_the_staging_slots_grew(ph, orc):
    """Later calls with more requests and tiles than a staging slot holds give
    the slots larger buffers; a captured call's replays keep theirs."""
    import torch
    k = 40
    ctx = ph.Context(0, max_instances=400)
    p, a = orc.lcg_params(64)
    n, e, _ = orc.seed(64, SEED + 4, k, (9, 17))
    s0 = np.arange(3, k + 3, dtype=np.uint64) * np.uint64(0x1234567890abc)
    ids = ctx.add_instances(64, n, e, s0=s0)
    starts = [ctx.get_state(int(i)) for i in ids]
    counts = 100 + np.arange(k) * 300
    reqs = _requests(ph, ids, counts)
    c = torch.empty(int(counts.sum()), dtype=torch.int64, device="cuda")
    want = [orc.generate(p, a, int(n[i]), int(e[i]), 0, int(s0[i]), int(counts[i]))[0] for i in range(k)]
    many = ctx.seed_instances(32, SEED + 5, 300, (9, 17), 0, 0)
    long = ctx.seed_instances(64, SEED + 6, 1, (9, 17), 0, 0)
    big = _requests(ph, np.concatenate([many[np.arange(9000) % 300], long]), [3] * 9000 + [(1 << 26) + (1 << 20)])
    room = torch.empty(27000 + (1 << 26) + (1 << 20), dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, capture_error_mode="relaxed"):
        ctx.generate(reqs, None, c, None, stream=torch.cuda.current_stream())
    for replay in range(3):
        c.fill_(-1)
        if replay:
            for i, (m, s, _, pos) in zip(ids, starts):
                ctx.set_state(int(i), m, s, pos)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        got = c.cpu().numpy().view(np.uint64)
        for i in range(k):
            compare_request(got, None, int(reqs["out_offset"][i]), int(counts[i]), want[i], None,
                            "replay %d, request %d" % (replay, i))
        for _ in range(9):
            ctx.generate(big, None, None, room)
        torch.cuda.synchronize()
    del graph
    ctx.close()
