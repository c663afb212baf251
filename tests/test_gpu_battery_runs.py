"""The runs test on blocks built of runs of chosen lengths, against the
oracle's counts (exact): runs of 19..23 around the last category, of 62..66
and 126..130 around one and two words, words without any change, a single
change in the block at every kind of place, and blocks whose last run is
long; and the report of large histograms with heavy cells."""

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


def _block(lengths):
    """A block of alternating runs of the given lengths (cycled, cut at M)."""
    bits = np.empty(M, dtype=bool)
    pos, v, i = 0, False, 0
    while pos < M:
        n = lengths[i % len(lengths)]
        bits[pos:pos + n] = v
        pos, v, i = pos + n, not v, i + 1
    return bits


def _single(at):
    bits = np.zeros(M, dtype=bool)
    bits[at:] = True
    return bits


BLOCKS = {
    "alternating": lambda: _block([1]),
    "19-23": lambda: _block([19, 20, 21, 22, 23, 1, 2]),
    "words": lambda: _block([62, 63, 64, 65, 66, 126, 127, 128, 129, 130, 7]),
    "long": lambda: _block([1, 5000, 3, 192, 64, 256]),
    "half": lambda: _block([M // 2]),
    "single early": lambda: _single(1),
    "single word edge": lambda: _single(64),
    "single word end": lambda: _single(63),
    "single last": lambda: _single(M - 1),
    "single last word": lambda: _single(M - 64),
    "two at the end": lambda: _single(M - 2) ^ _single(M - 1),
    "none": lambda: np.zeros(M, dtype=bool),
    "random": lambda: np.random.default_rng(5).random(M) < 0.5,
    "sparse": lambda: np.cumsum(np.random.default_rng(6).random(M) < 0.003) % 2 == 1,
}


@pytest.mark.parametrize("order", [1, -1])
def test_runs_of_chosen_lengths(ph, order):
    import torch
    names = list(BLOCKS)[::order]
    bat = ph.Battery(0)
    for name in names:
        r = np.where(BLOCKS[name](), 0.75, 0.25)
        bat.reset()
        bat.accumulate(torch.from_numpy(r).to("cuda:0"))
        got = bat.counts(ph.BATTERY_TESTS.index("runs")).astype(np.int64)
        assert np.array_equal(got, B.runs_counts(r)), name
    # all blocks in one sequence: no run crosses from one block to the next
    r = np.concatenate([np.where(BLOCKS[n](), 0.75, 0.25) for n in names])
    bat.reset()
    bat.accumulate(torch.from_numpy(r).to("cuda:0"))
    got = bat.counts(ph.BATTERY_TESTS.index("runs")).astype(np.int64)
    assert np.array_equal(got, B.runs_counts(r))
    # the same sequence has few distinct cells: chi^2 from heavy counts
    want = B.run_battery(r)
    rep = bat.report()
    for name in ("frequency", "serial2", "serial3", "serial4", "serial5"):
        assert rep[name][0] == pytest.approx(want[name][2], rel=1e-12), name
    bat.close()
