"""A call that finds no device memory is made again once torch has given back the
blocks that its allocator keeps for reuse (a pattern histogram leaves gigabytes
there); where torch has nothing to give or is capturing, and where memory is
still short, the error comes through.  Runs without a GPU: a stand-in for the
library answers."""

import pytest
import torch

import paper_1411_2484_amd as ph
from tests.test_binding_checks_cpu import FakeTensor


class ShortOfMemory:
    """Answers `fails` calls with PHPRNG_E_NOMEM, then PHPRNG_OK."""

    def __init__(self, fails):
        self.fails, self.calls, self.log = fails, 0, []

    def __getattr__(self, name):
        def call(*args):
            if name.endswith("_string") or name.endswith("_error"):
                return b"out of memory"
            if "destroy" in name:
                return ph.PHPRNG_OK
            self.log.append(name)
            self.calls += 1
            return ph.PHPRNG_E_NOMEM if self.calls <= self.fails else ph.PHPRNG_OK
        return call


def _generate():
    ctx = ph.Context.__new__(ph.Context)
    ctx._h, ctx.device = None, 0
    ctx.generate(ph.make_requests([0], [4], [0]), None, None, FakeTensor(torch.float64), stream=0)


CALLS = {"context": lambda: ph.Context(0), "battery": lambda: ph.Battery(0), "generate": _generate,
         "pattern": lambda: ph.pattern_histogram(ph.pattern_spec(4294967087, 9, 0, 1, 2, 4),
                                                 FakeTensor(torch.int64, device=None), 0)}


@pytest.mark.parametrize("call", list(CALLS))
@pytest.mark.parametrize("fails,initialized,capturing,made", [(1, True, False, 2), (2, True, False, 2),
                                                              (1, False, False, 1), (1, True, True, 1),
                                                              (0, True, False, 1)])
def test_made_again_after_torch_gave_back(monkeypatch, call, fails, initialized, capturing, made):
    short, given = ShortOfMemory(fails), []
    monkeypatch.setattr(ph, "lib", lambda: short)
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: initialized)
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: capturing)
    monkeypatch.setattr(torch.cuda, "empty_cache", lambda: given.append(short.calls))
    if fails >= made:
        with pytest.raises(ph.PhprngError) as ex:
            CALLS[call]()
        assert ex.value.status == ph.PHPRNG_E_NOMEM
    else:
        CALLS[call]()
    assert given == ([1] if made == 2 else []) and len(set(short.log)) == 1 and short.calls == made


@pytest.mark.parametrize("address,taken", [(0x10000, True), (0x10100, True), (0x10080, False), (0x10008, False)])
def test_scratch_at_an_address_that_the_library_refuses_is_not_taken(monkeypatch, address, taken):
    hist, block = FakeTensor(torch.int64), FakeTensor(torch.uint8)
    block.data_ptr = lambda: address
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(ph, "_stream_handle", lambda stream, device=None: 0)
    monkeypatch.setattr(torch, "empty", lambda *a, **k: block)
    got = ph._torch_scratch(ph.pattern_spec(4294967087, 9, 0, 1, 2, 4), hist, 0)
    assert got is (block if taken else None)
