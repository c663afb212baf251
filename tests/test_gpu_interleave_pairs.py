"""Interleaving moves two uniforms per access where counts are even and both
arrays lie at 16-byte addresses, one at a time elsewhere: even and odd numbers
of streams and lengths around whole tiles of 64, and arrays that start 8 bytes
past a 16-byte address; exact, with guards around the output."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("skew_in,skew_out", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("streams,length", [(64, 64), (64, 1024), (128, 66), (66, 130), (2, 2), (63, 64), (64, 63),
                                            (65, 129), (1, 1000), (1000, 1), (62, 192), (192, 62)])
def test_interleave_shapes_and_addresses(streams, length, skew_in, skew_out):
    import torch
    import paper_1411_2484_amd as ph
    n = streams * length
    src = torch.rand(n + 2, dtype=torch.float64, device="cuda")[skew_in:skew_in + n]
    buf = torch.full((n + 6,), -1.0, dtype=torch.float64, device="cuda")
    out = buf[2 + skew_out:2 + skew_out + n]
    assert src.data_ptr() % 16 == 8 * skew_in and out.data_ptr() % 16 == 8 * skew_out
    ph.interleave(src, out, streams, length)
    torch.cuda.synchronize()
    want = src.cpu().numpy().reshape(streams, length).T.ravel()
    assert np.array_equal(out.cpu().numpy(), want)
    rest = buf.cpu().numpy()
    assert (rest[:2 + skew_out] == -1).all() and (rest[2 + skew_out + n:] == -1).all()
