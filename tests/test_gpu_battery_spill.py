"""Scatter of the battery's histogram keys: whole tiles whose keys all fit
their buckets, tiles that meet a full bucket (uniforms crowded into one
partition of 2^15 cells until the room for a chunk of blocks runs out, in the
middle of a tile too), the shorter last tile of a block, and the values at the
ends of the bins; exact counts of the oracle.  And the time of each kernel
class, which runs from the kernel before it: the classes together take no
longer than the call on the host's clock (1% allowed for the two clocks)."""

import time

import numpy as np
import pytest

from oracle import battery as B

pytestmark = pytest.mark.gpu
M = 1 << 20


@pytest.fixture(scope="module")
def ph():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1411_2484_amd as ph
    ph.lib()
    return ph


def _uniforms(kind, blocks):
    rng = np.random.default_rng(blocks)
    r = rng.random(blocks * M)
    if kind == "crowded":
        r = r / 32 + 5 / 32
    elif kind == "half crowded":
        r = np.where(rng.random(r.size) < 0.6, r / 64 + 0.75, r)
    elif kind == "edges":
        r = rng.choice([0.0, 2.0 ** -53, 0.1, 0.5, np.nextafter(0.5, 1), 1 - 2.0 ** -53, 1.0, 0.99, 1 / 3], r.size)
    return r


@pytest.mark.parametrize("kind,blocks", [("uniform", 1), ("uniform", 3), ("edges", 2), ("crowded", 7),
                                         ("half crowded", 11)])
def test_histograms_with_full_buckets(ph, kind, blocks):
    import torch
    r = _uniforms(kind, blocks)
    bat = ph.Battery(0)
    d = torch.from_numpy(r).cuda()
    for call in range(2):
        bat.accumulate(d)
    want = {"frequency": B.frequency_counts(r), "poker": B.poker_counts(r)}
    for k in (2, 3, 4, 5):
        want["serial%d" % k] = B.serial_counts(r, k)
    for i, name in enumerate(ph.BATTERY_TESTS):
        if name in want:
            got = bat.counts(i)
            assert np.array_equal(np.asarray(got), 2 * np.asarray(want[name])), name
    assert set(want) <= set(ph.BATTERY_TESTS)
    bat.close()


def test_kernel_class_times(ph):
    import torch
    d = torch.rand(4 * M, dtype=torch.float64, device="cuda")
    bat = ph.Battery(0)
    torch.cuda.synchronize()
    t = time.perf_counter()
    for call in range(3):
        bat.accumulate(d)
    torch.cuda.synchronize()
    host_ms = (time.perf_counter() - t) * 1e3
    times = bat.timing()
    assert all(ms > 0 and n == 3 for ms, n in times.values())
    assert sum(ms for ms, _ in times.values()) <= 1.01 * host_ms
    bat.reset()
    assert all(ms == 0 and n == 0 for ms, n in bat.timing().values())
    bat.close()
