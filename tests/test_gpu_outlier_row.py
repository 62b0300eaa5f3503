"""Decoders' outlier row: the first 64 outliers of a chunk are read as one row
across the wavefront, further ones by rank.  Chunks with counts around the
row's length, at the chunk's ends and in a ragged last chunk must decode to
the oracle's bits, from LCQ1 and from packed streams (both are compared
exactly: a decode has one right result)."""
import numpy as np
import pytest

import oracle as O
import synth
from gpu_util import announce, bits, first_diff, gpu_decode

pytestmark = pytest.mark.gpu

EB = 1e-3


def _field(dt, q, count):
    """Four chunks and a ragged fifth, `count` NaNs in each: at the front, at
    the back, spread, alternating with values (as many as fit), and at the
    ragged end."""
    n = 4 * 1024 + 777
    x = synth.sines_1d(n, 77, dtype=dt)
    if q == "rel":
        x = np.abs(x) + dt(1.0)
    x[:count] = np.nan
    x[2 * 1024 - count:2 * 1024] = np.nan
    if count:
        x[2 * 1024 + (np.arange(count) * 1024) // count] = np.nan
        x[3 * 1024:3 * 1024 + min(2 * count, 1024):2] = np.nan
    m = min(count, n - 4 * 1024)
    x[n - m:] = np.nan
    return x


@pytest.mark.parametrize("dt", [np.float32, np.float64])
@pytest.mark.parametrize("q", ["abs", "rel"])
@pytest.mark.parametrize("count", [0, 1, 2, 63, 64, 65, 129, 1024])
def test_outlier_row_lengths(dt, q, count):
    import torch
    import paper_2407_15037_amd as lcq
    x = _field(dt, q, count)
    n = x.size
    st = O.quantize(q, x, EB)
    want = O.dequantize(st, dt, n)
    announce("outlier row", np.dtype(dt).name, q, count)
    got, status = gpu_decode(st, dt, n)
    assert status == lcq.OK
    assert first_diff(bits(got), bits(want)) is None
    buf = torch.from_numpy(O.pack(st, dt, n)).cuda()
    ws = torch.zeros(64, dtype=torch.uint8, device="cuda")
    tdt = torch.float32 if dt == np.float32 else torch.float64
    out = lcq.decompress(buf, tdt, n, ws=ws)
    assert lcq.stream_status(ws) == lcq.OK
    assert first_diff(bits(out.cpu().numpy()), bits(want)) is None
