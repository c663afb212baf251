"""GPU parity, bit for bit against the oracle, of the exponent chains at the
ends of the modulus ranges: width-32 moduli just above 2^31 and just below
2^32 (where the sign-free squarings and the negated messages leave the least
room) with every chain (3, 5, 9, 17, generic small ones, 65537, one above
2^31), under the pseudorandom and the constant skip, with the outputs c + R,
R alone and c alone, which are separate code paths."""

import random

import numpy as np
import pytest

from tests.gpu_helpers import alloc_outputs, compare_request, to_host

pytestmark = pytest.mark.gpu

EXPS = [3, 5, 9, 17, 7, 33, 65537, (1 << 31) + 11]
COUNT = 4500  # two whole tiles and a partial one


@pytest.fixture(scope="module")
def ph():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1411_2484_amd as ph
    ph.lib()
    return ph


def _moduli(orc, width):
    lo, hi = (1 << 31, 1 << 32) if width == 32 else (1 << 62, 1 << 63)
    out = []
    for start, step in ((lo + 1, 2), (hi - 1, -2)):
        n, got = start, 0
        while got < 4:
            if orc.is_prime(n):
                out.append(n)
                got += 1
            n += step
    return out


def _instances(orc, width):
    ns, es = [], []
    for n in _moduli(orc, width):
        for e in EXPS:
            if orc.check_instance(width, n, e) == 0:
                ns.append(n)
                es.append(e)
    assert set(es) >= {3, 5, 9, 17, 7, 65537}
    return ns, es


@pytest.mark.parametrize("width,sched", [(32, "skip"), (32, "constant"), (64, "constant")])
@pytest.mark.parametrize("outputs", ["c+R", "R", "c"])
def test_chains_at_the_range_ends(ph, orc, width, sched, outputs):
    rng = random.Random("%d %s %s" % (width, sched, outputs))
    p, a = orc.lcg_params(width)
    ns, es = _instances(orc, width)
    k = len(ns)
    m0 = [rng.choice([0, 1, n - 1, rng.randrange(n)]) for n in ns]
    ctx = ph.Context(0, max_instances=k)
    if sched == "skip":
        s0 = [rng.choice([1, p - 1, rng.randrange(1, p)]) for _ in ns]
        ids = ctx.add_instances(width, ns, es, m0=m0, s0=s0)
    else:
        b = [rng.choice([1, 2, n - 1, rng.randrange(1, n)]) for n in ns]
        ids = ctx.add_instances_skip(width, ns, es, b, m0=m0)
    want_c = outputs != "R"
    c32, c64, r = alloc_outputs(COUNT * k, want_c and width == 32, want_c and width == 64, outputs != "c")
    ctx.generate(ph.make_requests(ids, [COUNT] * k, np.arange(k, dtype=np.uint64) * COUNT), c32, c64, r)
    hc32, hc64, hr = to_host(c32, c64, r)
    got_c = hc32 if width == 32 else hc64
    for j, (n, e) in enumerate(zip(ns, es)):
        if sched == "skip":
            wc, wr, _, _ = orc.generate(p, a, n, e, m0[j], s0[j], COUNT)
        else:
            wc, wr = orc.generate_cskip(n, e, b[j], m0[j], COUNT)[:2]
        compare_request(got_c, hr, j * COUNT, COUNT, wc, wr,
                        "w%d %s n=%d e=%d" % (width, sched, n, e))
    ctx.close()
