"""Rows of a tile start at whole lines of the outputs: every offset of a
request modulo 32, with starts at the beginning, the end and inside of a tile
(at the end the shift moves all of the first tile's draws into the second),
lengths around tiles, chunks and single draws, requests packed against one
another so that a draw stored outside its request shows, and the last tiles
of a skip period.  Bit for bit against the oracle, both widths, both
schedules, every combination of outputs."""

import numpy as np
import pytest

from tests.gpu_helpers import alloc_outputs, compare_request, to_host

pytestmark = pytest.mark.gpu

P31 = (1 << 31) - 1
SEED = 0x14112484 + 5100


@pytest.fixture(scope="module")
def ph():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1411_2484_amd as ph
    ph.lib()
    return ph


def _starts_and_lengths(width, sched):
    tile = 2048 if width == 32 or sched == "constant" else 1024
    out = []
    for shift in range(32):
        for head in (0, 1, tile - 1, tile - 5, tile - 31, tile - 32, tile // 2 + 3 * shift):
            out.append((head, [1, 2, 40, tile - head, tile - head + 1, 3 * tile + 7 + shift][(shift + head) % 6]))
    # chunks of several tiles
    out += [(tile - 3, 9 * tile + 11), (5, 17 * tile), (tile - 31, 8 * tile + 33)]
    if width == 32 and sched == "skip":
        last = P31 - 1  # draws of a period
        out += [(last - 2046 - 5, 6000), (last - 3, 4100), (last - 1, 2), (last - 2046, 2046), (2 * last - 31, 40)]
    return out


@pytest.mark.parametrize("width,sched", [(32, "skip"), (32, "constant"), (64, "skip"), (64, "constant"),
                                         (64, "restored")])
@pytest.mark.parametrize("outputs", ["c+R", "R", "c"])
def test_every_offset_start_and_length(ph, orc, tab32, width, sched, outputs):
    cases = _starts_and_lengths(width, sched)
    k = len(cases)
    heads = np.array([h for h, _ in cases], dtype=np.uint64)
    counts = np.array([c for _, c in cases], dtype=np.uint64)
    # packed requests whose offsets run through all residues
    offs = np.concatenate([[0], np.cumsum(counts)[:-1]]).astype(np.uint64)
    assert len(set(int(o) % 32 for o in offs)) == 32
    n, e, _ = orc.seed(width, SEED + width, k, (9, 17, 3))
    p, a = orc.lcg_params(width)
    ctx = ph.Context(0, max_instances=k)
    if sched == "constant":
        ids = ctx.add_instances_skip(width, n, e, np.arange(1, k + 1, dtype=np.uint64), k0=heads)
    elif sched == "restored":
        s0 = np.arange(3, k + 3, dtype=np.uint64) * np.uint64(0x1234567890abc)
        ids = ctx.add_instances(width, n, e, s0=s0)
    else:
        ids = ctx.add_instances(width, n, e, k0=heads)
    ctx.set_tuning(tiles_per_chunk=4)
    want_c = outputs != "R"
    total = int(counts.sum())
    c32, c64, r = alloc_outputs(total, want_c and width == 32, want_c and width == 64, outputs != "c")
    ctx.generate(ph.make_requests(ids, counts, offs), c32, c64, r)
    hc32, hc64, hr = to_host(c32, c64, r)
    got_c = hc32 if width == 32 else hc64
    for i in range(k):
        h, cnt = int(heads[i]), int(counts[i])
        if sched == "constant":
            b = i + 1
            wc, wr, _ = orc.generate_cskip(int(n[i]), int(e[i]), b, h * b % int(n[i]), cnt)
        else:
            if sched == "restored":
                m, s = 0, int(s0[i])
            elif width == 32:
                m, s = orc.position(tab32, p, a, int(n[i]), 0, 1, h)
            else:
                m, s = orc.position(None, p, a, int(n[i]), 0, 1, h)
            wc, wr, _, _ = orc.generate(p, a, int(n[i]), int(e[i]), m, s, cnt)
        compare_request(got_c, hr, int(offs[i]), cnt, wc, wr,
                        "w%d %s start %d count %d offset %d" % (width, sched, h, cnt, int(offs[i])))
    ctx.close()
