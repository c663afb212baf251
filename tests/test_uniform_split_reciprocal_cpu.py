"""The kernels form R = (c+1)/(n+1) from a reciprocal in two parts, rcp =
RN(1/b) and rcp_lo = RN(1/b - rcp) with b = n + 1 (width 64: RN(n + 1)).

Width 32, integers 1 <= a < b <= 2^33: fma(a, rcp, RN(a rcp_lo)) is the IEEE
quotient (the sum before its one rounding is within 2^-105 of a/b, and a/b is
never within 2^-88 of a rounding boundary).  Width 64: the same value is
within one ulp of a/b, and one remainder-and-correct step with rcp rounds it
correctly (Markstein).  The tolerance is zero: every pair must give a / b.

The pairs, threads and hardest cases are those of csrc/recip_check.c; only
the two forms are replaced."""

import ctypes
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))

OLD32 = """  double q0 = a * y;
  double r = fma(-q0, b, a);
  return fma(r, y, q0);
"""
NEW32 = """  double yl = fma(-b, y, 1.0) / b;
  return fma(a, y, a * yl);
"""
OLD64 = """  double q0 = a * y;
  double q1 = fma(fma(-q0, b, a), y, q0);
  return fma(fma(-q1, b, a), y, q1);
"""
NEW64 = """  double yl = fma(-b, y, 1.0) / b;
  double q1 = fma(a, y, a * yl);
  return fma(fma(-q1, b, a), y, q1);
"""


@pytest.fixture(scope="module")
def rc(tmp_path_factory):
    src = open(os.path.join(HERE, "csrc", "recip_check.c")).read()
    assert src.count(OLD32) == 1 and src.count(OLD64) == 1
    d = tmp_path_factory.mktemp("rc2")
    path = str(d / "split.c")
    with open(path, "w") as f:
        f.write(src.replace(OLD32, NEW32).replace(OLD64, NEW64))
    out = str(d / "libsplit.so")
    subprocess.run(["gcc", "-O2", "-march=x86-64-v3", "-fno-fast-math", "-ffp-contract=off", "-fPIC", "-shared",
                    "-pthread", "-o", out, path, "-lm"], check=True)
    L = ctypes.CDLL(out)
    L.recip_exhaustive.restype = ctypes.c_uint64
    L.recip_exhaustive.argtypes = [ctypes.c_uint64] * 3 + [ctypes.c_int]
    L.recip_sampled.restype = ctypes.c_uint64
    L.recip_sampled.argtypes = [ctypes.c_uint64, ctypes.c_uint64, ctypes.c_int, ctypes.c_int,
                                ctypes.POINTER(ctypes.c_uint64)]
    return L


# mode: 0 / 1 width 32 random / near a midpoint; 2 / 3 / 4 width 64 random /
# near a midpoint / within ~2^-107 of one
@pytest.mark.parametrize("mode,pairs,least", [(0, 10 ** 8, 10 ** 8), (1, 2 * 10 ** 7, 10 ** 7),
                                              (2, 10 ** 8, 10 ** 8), (3, 2 * 10 ** 7, 10 ** 7),
                                              (4, 2 * 10 ** 6, 10 ** 6)])
def test_split_reciprocal_is_the_ieee_quotient(rc, mode, pairs, least):
    nt = max(1, min(os.cpu_count() or 1, 16))
    done = ctypes.c_uint64()
    bad = rc.recip_sampled(0x5711 + mode, (pairs + nt - 1) // nt, mode, nt, ctypes.byref(done))
    assert done.value >= least
    assert bad == 0


@pytest.mark.parametrize("b", [2 ** 31 + 12, 4294967088, 2 ** 32 - 4])
def test_split_reciprocal_every_numerator_at_both_ends(rc, b):
    nt = max(1, min(os.cpu_count() or 1, 16))
    assert rc.recip_exhaustive(b, 1, 1 << 22, nt) == 0
    assert rc.recip_exhaustive(b, b - (1 << 22), b, nt) == 0
