"""Constant-skip requests that end at the last positions below 2^64, where the
rows of the last tile, shifted to the lines of the outputs, run past 2^64: every
offset of a request modulo 32, ends and lengths around the last row, both
widths, every combination of outputs, bit for bit against the oracle."""

import numpy as np
import pytest

from tests.gpu_helpers import alloc_outputs, compare_request, to_host

pytestmark = pytest.mark.gpu

SEED = 0x14112484 + 6400
TOP = (1 << 64) - 1


@pytest.fixture(scope="module")
def ph():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1411_2484_amd as ph
    ph.lib()
    return ph


@pytest.mark.parametrize("width", [32, 64])
@pytest.mark.parametrize("outputs", ["c+R", "R", "c"])
def test_rows_at_the_last_positions(ph, orc, width, outputs):
    # (draws from the last position, draws asked for) at every offset mod 32
    ends = [(1, 1), (5, 4), (10, 10), (16, 1), (31, 30), (32, 32), (40, 3), (100, 100), (2047, 2047), (2100, 2099)]
    cases = [(back, count, off) for back, count in ends for off in range(32)]
    k = len(cases)
    counts = np.array([c for _, c, _ in cases], dtype=np.uint64)
    starts = np.array([TOP - b for b, _, _ in cases], dtype=np.uint64)
    room = np.cumsum([0] + [(int(c) + 63) // 32 * 32 for c in counts])
    offs = np.array([int(room[i]) + off for i, (_, _, off) in enumerate(cases)], dtype=np.uint64)
    n, e, _ = orc.seed(width, SEED + width, k, (9, 17, 3))
    b = np.arange(1, k + 1, dtype=np.uint64) * np.uint64(1234567)
    ctx = ph.Context(0, max_instances=k)
    ids = ctx.add_instances_skip(width, n, e, b, k0=starts)
    want_c = outputs != "R"
    out = alloc_outputs(int(room[-1]) + 64, want_c and width == 32, want_c and width == 64, outputs != "c")
    ctx.generate(ph.make_requests(ids, counts, offs), *out)
    hc32, hc64, hr = to_host(*out)
    for i, (back, count, off) in enumerate(cases):
        m = int(b[i]) * int(starts[i]) % int(n[i])
        wc, wr, _ = orc.generate_cskip(int(n[i]), int(e[i]), int(b[i]), m, count)
        compare_request(hc32 if width == 32 else hc64, hr, int(offs[i]), count, wc, wr,
                        "w%d %d draws, %d from the last position, offset %d" % (width, count, back, off))
    ctx.close()
