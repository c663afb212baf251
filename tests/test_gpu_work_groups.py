"""The persistent grid's work counters: a batch with few chunks per wave is
cut into groups with a counter each, one with at least ten chunks per wave
uses one counter.  Chunk counts around every edge (fewer chunks than waves,
one more than waves, groups of unequal size, the switch at ten per wave), three
calls in a row on the same context so that a counter left non-zero shows,
each compared bit for bit with the oracle."""

import numpy as np
import pytest

from tests.gpu_helpers import alloc_outputs, compare_request, to_host

pytestmark = pytest.mark.gpu

SEED = 0x14112484 + 4200


@pytest.fixture(scope="module")
def setup(orc):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1411_2484_amd as ph
    ph.lib()
    waves = torch.cuda.get_device_properties(0).multi_processor_count
    ctx = ph.Context(0, max_instances=64)
    yield ph, ctx, waves
    ctx.close()


@pytest.mark.parametrize("block,extra", [(64, -1), (64, 0), (64, 1), (64, 37), (64, 300), (64, "switch-1"),
                                         (64, "switch"), (64, "switch+7"), (256, 1), (256, 700)])
def test_chunk_counts_around_the_group_edges(setup, orc, block, extra):
    ph, ctx, cus = setup
    waves = cus * block // 64  # one block per CU, one tile per chunk
    if isinstance(extra, str):
        chunks = 10 * waves + int(extra[6:] or 0)
    else:
        chunks = waves + extra
    ctx.set_tuning(block_threads=block, blocks_per_cu=1, tiles_per_chunk=1, unroll=4)
    n, e, _ = orc.seed(32, SEED + block, 1, (9, 17))
    iid = int(ctx.add_instances(32, n, e)[0])
    p, a = orc.lcg_params(32)
    m, s = 0, 1
    count = chunks * 2048
    c32, _, r = alloc_outputs(count, True, False, True)
    for call in range(3):
        ctx.generate(ph.make_requests([iid], [count], [0]), c32, None, r)
        hc, _, hr = to_host(c32, None, r)
        wc, wr, m, s = orc.generate(p, a, int(n[0]), int(e[0]), m, s, count)
        compare_request(hc, hr, 0, count, wc, wr, "block %d, %d chunks, call %d" % (block, chunks, call))
