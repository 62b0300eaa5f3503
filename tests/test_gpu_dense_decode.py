"""Chunks with more outliers than one row of 64 holds: decoded to the oracle's
bits from LCQ1 streams, packed streams and a batch, with full and ragged
chunks of different counts side by side; and from streams whose chunk table
does not fit the sentinels, refused without a read past the outliers."""
import numpy as np
import pytest

import oracle as O
import synth
from gpu_util import announce, bits, first_diff, gpu_decode

pytestmark = pytest.mark.gpu

EB = 1e-3
COUNTS = [0, 64, 65, 200, 66, 127, 128, 129, 512, 3, 1023, 1024, 300]


def _field(dt, q):
    rng = np.random.default_rng(5)
    n = len(COUNTS) * 1024 - 301
    x = synth.sines_1d(n, 78, dtype=dt)
    if q == "rel":
        x = np.abs(x) + dt(1.0)
    for c, k in enumerate(COUNTS):
        v = x[c * 1024: (c + 1) * 1024]
        v[rng.permutation(v.size)[:k]] = np.nan
    return x


@pytest.mark.parametrize("dt", [np.float32, np.float64])
@pytest.mark.parametrize("q", ["abs", "rel", "noa"])
def test_dense_chunks(dt, q):
    import torch
    import paper_2407_15037_amd as lcq
    from paper_2407_15037_amd.batch import BatchPlan
    x = _field(dt, q)
    n = x.size
    st = O.quantize(q, x, EB)
    want = bits(O.dequantize(st, dt, n))
    announce("dense decode", np.dtype(dt).name, q)
    got, status = gpu_decode(st, dt, n)
    assert status == lcq.OK
    assert first_diff(bits(got), want) is None
    tdt = torch.float32 if dt == np.float32 else torch.float64
    ws = torch.zeros(64, dtype=torch.uint8, device="cuda")
    out = lcq.decompress(torch.from_numpy(O.pack(st, dt, n)).cuda(), tdt, n, ws=ws)
    assert lcq.stream_status(ws) == lcq.OK
    assert first_diff(bits(out.cpu().numpy()), want) is None
    plan = BatchPlan([{"x": torch.from_numpy(x).cuda(), "q": q, "eb": EB}])
    plan.quantize()
    plan.dequantize()
    assert plan.first_bad_field() == -1
    assert first_diff(bits(plan.fields[0]["out"].cpu().numpy()), want) is None


@pytest.mark.parametrize("dt", [np.float32, np.float64])
def test_wrong_chunk_table(dt):
    """A chunk's entry moved up by 100: the chunk before it looks dense, the
    values come from places that exist, and the stream is refused."""
    import paper_2407_15037_amd as lcq
    x = _field(dt, "abs")
    n, nch = x.size, len(COUNTS)
    st = O.quantize("abs", x, EB)
    k = int(st[16:24].view(np.uint64)[0])
    at = (64 + 4 * n + 15) // 16 * 16
    good = bits(O.dequantize(st, dt, n))
    for c, new in ((1, 100), (2, k - 1), (10, k), (12, k), (nch - 1, 0)):
        bad = st.copy()
        bad[at + 8 * c: at + 8 * c + 8] = np.frombuffer(np.uint64(new).tobytes(), np.uint8)
        announce("wrong chunk table", np.dtype(dt).name, c, new)
        got, status = gpu_decode(bad, dt, n)
        assert status == lcq.ERR_STREAM
        same = np.ones(nch, bool)
        same[c - 1: c + 1] = False
        for i in np.flatnonzero(same):  # chunks that the entry does not concern
            sl = slice(i * 1024, (i + 1) * 1024)
            assert first_diff(bits(got)[sl], good[sl]) is None, i
