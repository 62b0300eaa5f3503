"""Where quantize and compress change their route: one workgroup for small
fields (the limits differ by dtype and quantizer), pass-1 workgroups' totals
or atomic group sums.  Streams at and just past each limit must equal the oracle's
byte for byte, with output and workspace full of garbage before the call,
with outliers in smooth data, in every value, and with no finite value at
all (NOA's empty range)."""
import numpy as np
import pytest

import oracle as O
import synth
from gpu_util import announce, first_diff

pytestmark = pytest.mark.gpu


def _gpu_stream(q, x, eb):
    import torch
    import paper_2407_15037_amd as lcq
    xt = torch.from_numpy(x).cuda()
    ws = torch.full((lcq.workspace_bytes(q, xt.dtype, x.size),), 0xA5, dtype=torch.uint8,
                    device="cuda")
    out = torch.full((lcq.max_stream_bytes(xt.dtype, x.size),), 0x5A, dtype=torch.uint8,
                     device="cuda")
    buf, nb = lcq.quantize(xt, q, eb, out=out, ws=ws)
    return buf[: int(nb.item())].cpu().numpy()


def _data(kind, dt, n, q, eb):
    x = synth.sines_1d(n, n % 1000, dtype=dt)
    if kind == "nan":
        return np.full(n, np.nan, dt)
    if kind == "bits":
        ub = np.uint64 if dt == np.float64 else np.uint32
        return np.random.default_rng(n).integers(0, np.iinfo(ub).max, n, dtype=ub).view(dt)
    if q == "noa":
        return synth.with_specials(x, "noa", max(19, n // 300), 3, eb)
    x, _, _ = synth.inject_specials(x, max(19, n // 300), 3, eb)
    return x


@pytest.mark.parametrize("dt", [np.float32, np.float64])
@pytest.mark.parametrize("q", ["abs", "rel", "noa"])
@pytest.mark.parametrize("n", [1, 3, 1024, 1025, 16 * 1024, 16 * 1024 + 1, 18 * 1024,
                               18 * 1024 + 1, 24 * 1024 - 5, 24 * 1024 + 1, 32 * 1024,
                               32 * 1024 + 1])
def test_small_field_limits(dt, q, n):
    for kind in ("smooth", "bits", "nan"):
        x = _data(kind, dt, n, q, 1e-3)
        announce("small field", np.dtype(dt).name, q, n, kind)
        assert first_diff(_gpu_stream(q, x, 1e-3), O.quantize(q, x, 1e-3)) is None, kind


# 4096 pass-1 workgroups of 8 (float32 REL) or 4 chunks, and one more
@pytest.mark.parametrize("q,dt,n", [("rel", np.float32, 4096 * 8 * 1024),
                                    ("rel", np.float32, 4096 * 8 * 1024 + 1),
                                    ("abs", np.float32, 4096 * 4 * 1024),
                                    ("abs", np.float32, 4096 * 4 * 1024 + 1),
                                    ("abs", np.float64, 4096 * 4 * 1024),
                                    ("abs", np.float64, 4096 * 4 * 1024 + 1)])
def test_totals_limit(q, dt, n):
    x = synth.sines_1d(n, 11, dtype=dt)
    x[::977] = np.nan              # about one per chunk
    x[n // 2: n // 2 + 40 * 1024: 9] = np.nan    # 114 per chunk
    x[n // 4: n // 4 + 300 * 1024: 3] = np.nan   # 342 per chunk: over either stage cap
    x[n - 700:] = np.nan
    announce("totals limit", q, np.dtype(dt).name, n)
    assert first_diff(_gpu_stream(q, x, 1e-3), O.quantize_mt(q, x, 1e-3)) is None


# compress: 2048 workgroups of 4 chunks, and one more
@pytest.mark.parametrize("dt", [np.float32, np.float64])
@pytest.mark.parametrize("n", [2048 * 4 * 1024, 2048 * 4 * 1024 + 1])
def test_compress_totals_limit(dt, n):
    import torch
    import paper_2407_15037_amd as lcq
    x = synth.sines_1d(n, 12, dtype=dt)
    x[::977] = np.nan
    x[n // 4: n // 4 + 300 * 1024: 3] = np.nan
    x[n // 2: n // 2 + 5 * 1024] = np.nan   # whole chunks
    x[n - 700:] = np.nan
    announce("compress totals limit", np.dtype(dt).name, n)
    xt = torch.from_numpy(x).cuda()
    ws = torch.full((lcq.compress_workspace_bytes("abs", xt.dtype, n),), 0xA5, dtype=torch.uint8,
                    device="cuda")
    out = torch.full((lcq.pack_max_bytes(xt.dtype, n),), 0x5A, dtype=torch.uint8, device="cuda")
    pk, nb = lcq.compress(xt, "abs", 1e-3, out=out, ws=ws)
    want = O.pack(O.quantize_mt("abs", x, 1e-3), dt, n)
    assert first_diff(pk[: int(nb.item())].cpu().numpy(), want) is None


# NOA: 512 range workgroups of 8192 float32 / 4096 float64 values, and one more
@pytest.mark.parametrize("dt,n", [(np.float32, 512 * 8192), (np.float32, 512 * 8192 + 1),
                                  (np.float64, 512 * 4096), (np.float64, 512 * 4096 + 1),
                                  (np.float32, 64 * 8192 + 1)])
def test_noa_fold_limit(dt, n):
    import torch
    import paper_2407_15037_amd as lcq
    x = synth.with_specials(synth.sines_1d(n, 13, dtype=dt), "noa", n // 500, 5, 1e-3)
    x[-1] = dt(3.0) * np.abs(x[np.isfinite(x)]).max()  # the range ends in the last workgroup
    announce("noa fold limit", np.dtype(dt).name, n)
    st = O.quantize_mt("noa", x, 1e-3)
    assert first_diff(_gpu_stream("noa", x, 1e-3), st) is None
    pk, nb = lcq.compress(torch.from_numpy(x).cuda(), "noa", 1e-3)
    assert first_diff(pk[: int(nb.item())].cpu().numpy(), O.pack(st, dt, n)) is None


# pack: 2048 plan workgroups of 8 chunks, and one more; a small ragged one
@pytest.mark.parametrize("n", [1, 4 * 1024 + 1, 8 * 1024 + 1, 2048 * 8 * 1024, 2048 * 8 * 1024 + 1])
def test_pack_totals_limit(n):
    import torch
    import paper_2407_15037_amd as lcq
    x = synth.sines_1d(n, 14, dtype=np.float32)
    x[::977] = np.nan
    st = O.quantize_mt("abs", x, 1e-3)
    announce("pack totals limit", n)
    ws = torch.full((lcq.pack_workspace_bytes(torch.float32, n),), 0xA5, dtype=torch.uint8,
                    device="cuda")
    out = torch.full((lcq.pack_max_bytes(torch.float32, n),), 0x5A, dtype=torch.uint8, device="cuda")
    pk, nb = lcq.pack(torch.from_numpy(st).cuda(), torch.float32, n, out=out, ws=ws)
    assert lcq.stream_status(ws) == lcq.OK
    assert first_diff(pk[: int(nb.item())].cpu().numpy(), O.pack(st, np.float32, n)) is None


# bin widths from subnormal to near the largest value: their reciprocals
# overflow, are subnormal, or round at the ends of the range
@pytest.mark.parametrize("dt,exps", [(np.float32, (-37, -30, 0, 30, 38)),
                                     (np.float64, (-306, -300, 0, 300, 308))])
@pytest.mark.parametrize("n", [5000, 40000])
def test_noa_scales(dt, exps, n):
    for e in exps:
        for eb in (0.3, 1e-2, 1e-7):
            x = synth.sines_1d(n, 15, dtype=np.float64)
            x = (x / np.abs(x).max() * 10.0 ** e).astype(dt)
            announce("noa scales", np.dtype(dt).name, n, e, eb)
            assert first_diff(_gpu_stream("noa", x, eb), O.quantize("noa", x, eb)) is None, (e, eb)
