"""Collision trials, which workgroups take in turn with the next trial's
uniforms already loaded: fewer trials than workgroups, one round, a round and
a part of the next, several calls; random uniforms, uniforms crowded into few
urns, and equal ones (every ball but the first a collision).  Exact counts of
the oracle."""

import numpy as np
import pytest

from oracle import battery as B

pytestmark = pytest.mark.gpu
M = 1 << 20


@pytest.mark.parametrize("blocks", [1, 4, 5, 9])
@pytest.mark.parametrize("kind", ["random", "crowded", "equal", "mixed"])
def test_collision_counts(kind, blocks):
    import torch
    import paper_1411_2484_amd as ph
    r = np.random.default_rng(blocks).random(blocks * M)
    if kind == "crowded":
        r = np.floor(r * 40000) / (1 << 20)
    elif kind == "equal":
        r[:] = 1.0
    elif kind == "mixed":  # trials of very different counts next to one another
        r = np.where((np.arange(r.size) // (1 << 14)) % 3 == 0, r, r / 7)
    bat = ph.Battery(0)
    d = torch.from_numpy(r).cuda()
    for call in range(2):
        bat.accumulate(d)
    got = np.asarray(bat.counts(ph.BATTERY_TESTS.index("collision")))
    assert np.array_equal(got, 2 * np.asarray(B.collision_counts(r)))
    bat.close()
