"""Performance cases of the generator: what a user's program has it do.

Each case is one pass through the package's public entry points (Context,
Graph, Battery, interleave, pattern_*), on instances that are seeded and
positioned beforehand, with the library's default launch shapes.  A pass of a
generation case continues every stream where the last one left it, as a
program's next call does.

Kinds and the ranges that draw() covers:
  one      one width-32 stream, 10^2 .. 4 10^6 draws per call
  serve    the batches of the serving loop: 1 .. 2048 requests of log-uniform
           length in [2^8, 2^20] on resident instances, 90% width 32, uniforms
           only, per-call timing off
  batch    equal requests on many width-32 streams, uniforms or uniforms and
           ciphertexts, even and odd lengths
  ragged   streams of log-uniform length in [2^10, 2^22] at starts in
           [0, 2^40), ciphertexts and uniforms
  mixed    width-64 and width-32 streams in one call, ciphertexts and uniforms
  w64      width-64 streams restored from an arbitrary state (m, s), which
           lies beyond the positioning table
  counter  constant-skip streams of both widths (the counter mode)
  graph    repeat draws of a small fixed batch from a captured graph
  battery  the nine statistical tests on a sequence of uniforms, as they come
           or interleaved over streams first
  pattern  the full-period pattern over a slice of the skips
"""

import math

import numpy as np
import torch

import paper_1411_2484_amd as ph

P32, A32 = (1 << 31) - 1, 784588716
P64, A64 = (1 << 61) - 1, 1633150009242682173
E_USUAL = (9, 17)


def listed():
    return [
        # the shortest call: a simulation that refills a small buffer from its stream
        {"name": "one_small", "kind": "one", "draws": 1000, "c": False},
        # 10^6 draws of one stream with its ciphertexts, the single-stream workload
        {"name": "one_stream", "kind": "one", "draws": 1000000, "c": True},
        # a serving batch under light load: two requests
        {"name": "serve_light", "kind": "serve", "requests": 2, "resident": 20000},
        # a serving batch near saturation
        {"name": "serve_full", "kind": "serve", "requests": 1024, "resident": 20000},
        # a repeated small refill of 64 streams from a captured graph
        {"name": "graph_small", "kind": "graph", "streams": 64, "draws": 4096},
        # the headline batch: 4096 streams x 2^18 uniforms
        {"name": "batch_uniforms", "kind": "batch", "streams": 4096, "draws": 1 << 18, "c": False},
        # streams of very different lengths and starts, ciphertexts and uniforms
        {"name": "ragged_both", "kind": "ragged", "streams": 2048, "lo": 10, "hi": 22},
        # both widths in one call
        {"name": "mixed_widths", "kind": "mixed", "n64": 256, "n32": 256, "draws": 1 << 20},
        # width-64 streams restored from saved states, odd length
        {"name": "w64_restored", "kind": "w64", "streams": 200, "draws": 300007, "c": False},
        # the counter mode of both widths, odd length
        {"name": "counter_mode", "kind": "counter", "n64": 500, "n32": 1000, "draws": 100003, "c": True},
        # the battery on 64 interleaved streams of 2^20 uniforms
        {"name": "battery_interstream", "kind": "battery", "blocks": 64, "streams": 64},
        # a slice of the three-point pattern of the published example instance
        {"name": "pattern_slice", "kind": "pattern", "dim": 3, "bins": 4096, "l0": 4, "skips": (1 << 27) + 12345},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["one", "serve", "batch", "ragged", "mixed", "w64", "counter", "graph", "battery", "pattern"])
    if kind == "one":
        return {"kind": kind, "draws": _log(rng, 100, 4000000), "c": rng.random() < 0.5}
    if kind == "serve":
        return {"kind": kind, "requests": _log(rng, 1, 2048), "resident": _log(rng, 1000, 50000)}
    if kind == "batch":
        streams = _log(rng, 2, 8192)
        return {"kind": kind, "streams": streams, "draws": _log(rng, 500, min(1 << 22, (1 << 29) // streams)),
                "c": rng.random() < 0.5}
    if kind == "ragged":
        return {"kind": kind, "streams": _log(rng, 16, 1024), "lo": 10, "hi": rng.randint(14, 22)}
    if kind == "mixed":
        n64, n32 = _log(rng, 1, 600), _log(rng, 1, 600)
        return {"kind": kind, "n64": n64, "n32": n32,
                "draws": _log(rng, 200, min(1 << 21, (1 << 28) // (n64 + n32)))}
    if kind == "w64":
        streams = _log(rng, 1, 300)
        return {"kind": kind, "streams": streams, "draws": _log(rng, 300, min(1 << 21, (1 << 27) // streams)),
                "c": rng.random() < 0.5}
    if kind == "counter":
        n64, n32 = _log(rng, 1, 1000), _log(rng, 1, 2000)
        return {"kind": kind, "n64": n64, "n32": n32,
                "draws": _log(rng, 200, min(1 << 21, (1 << 28) // (n64 + n32))), "c": rng.random() < 0.5}
    if kind == "graph":
        return {"kind": kind, "streams": _log(rng, 1, 1024), "draws": _log(rng, 200, 20000)}
    if kind == "battery":
        blocks = _log(rng, 1, 100)
        return {"kind": kind, "blocks": blocks, "streams": blocks if rng.random() < 0.5 else 0}
    dim = rng.choice([2, 3, 4, 5])
    bins = {2: 1 << 20, 3: rng.choice([1000, 4096]), 4: rng.choice([100, 256]), 5: rng.choice([33, 64])}[dim]
    return {"kind": kind, "dim": dim, "bins": bins, "l0": rng.randint(1, 8), "skips": _log(rng, 1 << 20, 1 << 26)}


# ---- inputs from the seed -------------------------------------------------------


def _counts(case):
    """Request lengths: part of the case where they are log-uniform, so that
    every seed of a case asks for the same sizes."""
    rng = np.random.default_rng([case.get("requests", 0), case.get("streams", 0), case.get("hi", 0)])
    if case["kind"] == "serve":
        return np.floor(2.0 ** (8 + 12 * rng.random(case["requests"]))).astype(np.uint64)
    if case["kind"] == "ragged":
        lo, hi = case["lo"], case["hi"]
        return np.floor(2.0 ** (lo + (hi - lo) * rng.random(case["streams"]))).astype(np.uint64)
    n = case.get("streams", 0) or case.get("n64", 0) + case.get("n32", 0) or 1
    return np.full(n, case["draws"], dtype=np.uint64)


def _offsets(counts):
    return np.concatenate([[0], np.cumsum(counts)[:-1]]).astype(np.uint64)


def _arrays(total, c32, c64):
    r = torch.empty(total, dtype=torch.float64, device="cuda")
    a = torch.zeros(total, dtype=torch.int32, device="cuda") if c32 else None
    b = torch.zeros(total, dtype=torch.int64, device="cuda") if c64 else None
    return a, b, r


def _skips(width, seed, count):
    """Constant skips b in [1, 2^30] of the counter mode."""
    rng = np.random.default_rng([seed, width, 2])
    b = rng.integers(1, 1 << 30, count).astype(np.uint64)
    b[::2] = 1  # the unit skip is the usual one
    return b


def _states64(seed, count):
    """Saved states (m, s) of width-64 streams, anywhere in the period."""
    rng = np.random.default_rng([seed, 3])
    return (rng.integers(0, 1 << 62, count).astype(np.uint64), rng.integers(1, P64, count).astype(np.uint64))


def _tested(case, seed):
    """The sequence that the battery tests: uniforms in (0, 1) on a grid of 2^-32."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    n = case["blocks"] << 20
    return (torch.randint(0, 1 << 32, (n,), generator=g, device="cuda").to(torch.float64) + 1) / 4294967297.0


def prepare(case, seed):
    kind = case["kind"]
    state = {"kind": kind}
    if kind == "battery":
        state["r"] = _tested(case, seed)
        state["streams"] = case["streams"]
        state["mixed"] = torch.empty_like(state["r"]) if case["streams"] else None
        state["battery"] = ph.Battery(0)
        return state
    if kind == "pattern":
        lo = 1 + seed * 7919 % (P32 - 1 - case["skips"])
        state["spec"] = ph.pattern_spec(4294967087, 9, seed % 1000003, case["l0"], case["dim"], case["bins"], lo,
                                        lo + case["skips"])
        state["hist"] = torch.zeros(case["bins"] ** (case["dim"] - 1), dtype=torch.int64, device="cuda")
        return state
    counts = _counts(case)
    total = int(counts.sum())
    c32 = c64 = False
    if kind in ("one", "batch", "graph"):
        ctx = ph.Context(0, max_instances=len(counts))
        ids = ctx.seed_instances(32, seed, len(counts), E_USUAL, 0, 0)
        c32 = case.get("c", False)
    elif kind == "ragged":
        ctx = ph.Context(0, max_instances=len(counts))
        ids = ctx.seed_instances(32, seed, len(counts), E_USUAL, 0, 1 << 40)
        c32 = True
    elif kind == "serve":
        n = case["resident"]
        ctx = ph.Context(0, max_instances=n)
        a = ctx.seed_instances(32, seed, n - n // 10, E_USUAL, 0, 1 << 40)
        b = ctx.seed_instances(64, seed + 1, n // 10, E_USUAL, 0, 1 << 32)
        rng = np.random.default_rng([seed, 4])
        ids = np.concatenate([a, b])[rng.integers(0, n, len(counts))]
        ctx.set_timing(False)
    elif kind == "mixed":
        ctx = ph.Context(0, max_instances=len(counts))
        ids = np.concatenate([ctx.seed_instances(64, seed, case["n64"], E_USUAL, 0, 0),
                              ctx.seed_instances(32, seed + 1, case["n32"], E_USUAL, 0, 0)])
        c32 = c64 = True
    elif kind == "w64":
        n, e, _ = ph.phprng_draw_instances(64, seed, len(counts), E_USUAL)
        m, s = _states64(seed, len(counts))
        ctx = ph.Context(0, max_instances=len(counts))
        ids = ctx.add_instances(64, n, e, m0=m, s0=s)
        c64 = case["c"]
    else:  # counter
        ctx = ph.Context(0, max_instances=len(counts))
        ids = []
        for w, k, sd in ((64, case["n64"], seed), (32, case["n32"], seed + 1)):
            n, e, _ = ph.phprng_draw_instances(w, sd, k, E_USUAL)
            ids.append(ctx.add_instances_skip(w, n, e, _skips(w, sd, k)))
        ids = np.concatenate(ids)
        c32 = c64 = case["c"]
    state["ctx"] = ctx
    state["requests"] = ph.make_requests(ids, counts, _offsets(counts))
    state["c32"], state["c64"], state["r"] = _arrays(total, c32, c64)
    if kind == "graph":
        state["graph"] = ctx.graph(state["requests"], None, None, state["r"])
    return state


# ---- one pass ----------------------------------------------------------------------

_SMALL_TESTS = ("poker", "collision", "runs", "fourier")


def run(state):
    if state["kind"] == "battery":
        bat, r = state["battery"], state["r"]
        bat.reset()
        if state["streams"]:
            ph.interleave(r, state["mixed"], state["streams"], r.numel() // state["streams"])
            r = state["mixed"]
        bat.accumulate(r)
        out = {"report": bat.report()}
        for t in _SMALL_TESTS:
            out[t] = bat.counts(ph.BATTERY_TESTS.index(t))
        return out
    if state["kind"] == "pattern":
        state["hist"].zero_()
        ph.pattern_histogram(state["spec"], state["hist"])
        return {"hist": state["hist"], "chi2": ph.pattern_chi2(state["spec"], state["hist"])}
    if "graph" in state:
        state["graph"].launch()
    else:
        state["ctx"].generate(state["requests"], state["c32"], state["c64"], state["r"])
    return {"c32": state["c32"], "c64": state["c64"], "r": state["r"]}


def work(case):
    """Outputs written once (and the battery's sequence read once); the
    floating-point operations of the battery's transforms."""
    kind = case["kind"]
    if kind == "battery":
        n = case["blocks"] << 20
        moved = 2 * n if case["streams"] else 0
        return {"bytes": 8 * (n + moved), "flops": 2.5 * n * 20}
    if kind == "pattern":
        cells = case["bins"] ** (case["dim"] - 1)
        return {"bytes": 8 * 3 * cells, "flops": 0}
    if kind in ("serve", "ragged"):
        total = int(_counts(case).sum())
    else:
        total = int(_counts(case).size) * case["draws"]
    if kind == "ragged":
        return {"bytes": 12 * total, "flops": 0}
    if kind == "mixed":
        return {"bytes": (16 * case["n64"] + 12 * case["n32"]) * case["draws"], "flops": 0}
    if kind == "counter":
        c = case["c"]
        return {"bytes": (case["n64"] * (16 if c else 8) + case["n32"] * (12 if c else 8)) * case["draws"],
                "flops": 0}
    per = 8 + ((8 if kind == "w64" else 4) if case.get("c") else 0)
    return {"bytes": per * total, "flops": 0}


# ---- the same in plain Python and numpy ----------------------------------------------

_M64 = (1 << 64) - 1


def _prime(n, bases):
    for q in (3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37):
        if n % q == 0:
            return False
    d, s = n - 1, 0
    while d % 2 == 0:
        d, s = d // 2, s + 1
    for a in bases:
        x = pow(a, d, n)
        if x in (1, n - 1):
            continue
        for _ in range(s - 1):
            x = x * x % n
            if x == n - 1:
                break
        else:
            return False
    return True


def _draw_instances(width, seed, count, k_lo, k_hi):
    """The seeded draw of (n, e, k) that phprng.h documents."""
    state = seed & _M64
    lo = span = 1 << (31 if width == 32 else 62)
    bases = (2, 3, 5, 7, 11) if width == 32 else (2, 3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37)

    def step():
        nonlocal state
        state = (state + 0x9E3779B97F4A7C15) & _M64
        z = state
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9 & _M64
        z = (z ^ (z >> 27)) * 0x94D049BB133111EB & _M64
        return z ^ (z >> 31)

    seen, out = set(), []
    while len(out) < count:
        n = (lo + step() % span) | 1
        if n in seen or not _prime(n, bases):
            continue
        y = step()
        e = next((E_USUAL[(y + t) % 2] for t in range(2) if math.gcd(E_USUAL[(y + t) % 2], n - 1) == 1), None)
        if e is None:
            continue
        seen.add(n)
        out.append((n, e, k_lo + step() % (k_hi - k_lo) if k_hi > k_lo else k_lo))
    return out


def _stream(width, n, e, m, s, count):
    """Algorithm (9) from (m, s), step by step."""
    p, a = (P32, A32) if width == 32 else (P64, A64)
    c = np.empty(count, dtype=np.uint64)
    for i in range(count):
        s = s * a % p
        m = (m + s) % n
        c[i] = pow(m, e, n)
    return c


def _counter_stream(n, e, b, count):
    c = np.empty(count, dtype=np.uint64)
    m = 0
    for i in range(count):
        m = (m + b) % n
        c[i] = pow(m, e, n)
    return c


def _chi2(keys, cells):
    o = np.bincount(keys, minlength=cells).astype(np.float64)
    ex = keys.size / cells
    return float(((o - ex) ** 2 / ex).sum())


def _exact_battery(case, seed):
    r = _tested(case, seed).cpu().numpy()
    if case["streams"]:
        r = r.reshape(case["streams"], -1).T.copy().reshape(-1)
    blocks = r.reshape(-1, 1 << 20)
    report = {}
    for name, dim, bins in (("frequency", 1, 1 << 20), ("serial2", 2, 1024), ("serial3", 3, 100),
                            ("serial4", 4, 32), ("serial5", 5, 16)):
        use = (1 << 20) // dim * dim
        b = np.minimum((blocks[:, :use] * bins).astype(np.int64), bins - 1).reshape(-1, dim)
        key = np.zeros(b.shape[0], dtype=np.int64)
        for i in range(dim):
            key = key * bins + b[:, i]
        report[name] = (_chi2(key, bins ** dim), None, None, None)
    return {"report": report}


def exact(case, seed):
    """Outputs of the first pass in 64 bits; None where plain Python would
    take too long or the start is far from the base state."""
    kind = case["kind"]
    if kind == "battery":
        return _exact_battery(case, seed) if case["blocks"] <= 64 else None
    if kind in ("pattern", "serve", "ragged"):
        return None
    counts = _counts(case)
    if int(counts.sum()) > 4000000:
        return None
    n_streams = len(counts)
    runs = []  # (width, n, e, ciphertexts)
    if kind in ("one", "batch", "graph"):
        for n, e, _ in _draw_instances(32, seed, n_streams, 0, 0):
            runs.append((32, n, _stream(32, n, e, 0, 1, case["draws"])))
    elif kind == "mixed":
        for w, k, sd in ((64, case["n64"], seed), (32, case["n32"], seed + 1)):
            for n, e, _ in _draw_instances(w, sd, k, 0, 0):
                runs.append((w, n, _stream(w, n, e, 0, 1, case["draws"])))
    elif kind == "w64":
        m, s = _states64(seed, n_streams)
        for (n, e, _), m0, s0 in zip(_draw_instances(64, seed, n_streams, 0, 0), m, s):
            runs.append((64, n, _stream(64, n, e, int(m0), int(s0), case["draws"])))
    else:
        for w, k, sd in ((64, case["n64"], seed), (32, case["n32"], seed + 1)):
            for (n, e, _), b in zip(_draw_instances(w, sd, k, 0, 0), _skips(w, sd, k)):
                runs.append((w, n, _counter_stream(n, e, int(b), case["draws"])))
    r = np.concatenate([(c + np.uint64(1)).astype(np.float64) / float(n + 1) for _, n, c in runs])
    out = {"r": r, "c32": None, "c64": None}
    has = {32: case.get("c", False) and kind in ("one", "batch", "counter") or kind == "mixed",
           64: case.get("c", False) and kind in ("w64", "counter") or kind == "mixed"}
    for width, key, dtype in ((32, "c32", np.uint32), (64, "c64", np.uint64)):
        if has[width]:
            c = np.concatenate([c if w == width else np.zeros_like(c) for w, _, c in runs])
            out[key] = c.astype(dtype).view(np.int32 if width == 32 else np.int64)
    return out
