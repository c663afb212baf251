"""The pattern histogram with caller-owned scratch: the same counts on torch's
current stream (torch's memory) and on another stream (the library's own),
scratch that is reused between calls, refused scratch, and the bins at the
ends of their range (1, 2, 2^24, and a prime count), against the oracle."""

import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

P31, A31, N = (1 << 31) - 1, 784588716, 4294967087


@pytest.fixture(scope="module")
def ph():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1411_2484_amd as ph
    ph.lib()
    return ph


@pytest.mark.parametrize("dim,bins", [(2, 1), (2, 2), (2, 1 << 24), (2, 16777213), (3, 1), (3, 4093), (4, 255),
                                      (5, 63)])
@pytest.mark.parametrize("where", ["current", "other"])
def test_scratch_of_both_kinds_gives_the_oracle_counts(ph, orc, dim, bins, where):
    import torch
    args = (N, 9, 3, 2, dim, bins)
    s_lo, s_hi = 5000, 5000 + 33000
    spec = ph.pattern_spec(*args, s_lo, s_hi)
    hist = torch.zeros(bins ** (dim - 1), dtype=torch.int64, device="cuda:0")
    torch.cuda.synchronize()
    stream = torch.cuda.Stream() if where == "other" else None
    for _ in range(2):  # counts add up; the second call reuses freed scratch
        ph.pattern_histogram(spec, hist, stream)
    want = 2 * orc.pattern_hist(N, 9, P31, A31, 3, 2, dim, bins, s_lo, s_hi).astype(np.int64)
    assert np.array_equal(hist.cpu().numpy(), want)


def test_refused_scratch(ph):
    import torch
    spec = ph.pattern_spec(N, 9, 0, 1, 3, 16, 1, 1000)
    L, ref = ph.lib(), ctypes.byref
    need = ctypes.c_uint64()
    assert L.phprng_pattern_workspace(ref(spec), ref(need)) == ph.PHPRNG_OK
    assert L.phprng_pattern_workspace(ref(spec), None) == ph.PHPRNG_E_INVALID
    bad = ph.pattern_spec(N, 9, 0, 1, 6, 16, 1, 1000)
    assert L.phprng_pattern_workspace(ref(bad), ref(need)) == ph.PHPRNG_E_INVALID
    hist = torch.zeros(256, dtype=torch.int64, device="cuda:0")
    ws = torch.empty(need.value + 256, dtype=torch.uint8, device="cuda:0")
    st = torch.cuda.current_stream().cuda_stream
    for ptr, size, status in ((None, need.value, ph.PHPRNG_E_INVALID), (ws.data_ptr() + 8, need.value,
                              ph.PHPRNG_E_INVALID), (ws.data_ptr(), need.value - 1, ph.PHPRNG_E_RANGE)):
        assert L.phprng_pattern_histogram_ws(ref(spec), hist.data_ptr(), ptr, size, st) == status
    assert L.phprng_pattern_histogram_ws(ref(spec), None, ws.data_ptr(), need.value, st) == ph.PHPRNG_E_INVALID
    torch.cuda.synchronize()
    assert int(hist.sum()) == 0
    assert L.phprng_pattern_histogram_ws(ref(spec), hist.data_ptr(), ws.data_ptr(), need.value, st) == ph.PHPRNG_OK
    assert int(hist.sum()) == 999
