"""Quantize pass 2 where a stretch of hard data lies in a smooth field: groups
of chunks with far more outliers than the average one, that hold short rows
(1 to 32 outliers), longer ones (33 to the stage cap, the cap itself among
them) and chunks over the cap side by side, the field's ragged last chunk
among them; and such chunks in groups that are not hot.  With totals per
first-pass workgroup and with sums per group; alone and in a batch.  The
oracle's own counts show that the inputs are what they are meant to be."""
import numpy as np
import pytest

import oracle as O
import synth
from gpu_util import announce, first_diff

CHUNK = 1024
CAP = {np.float32: 128, np.float64: 256}
EB = 1e-3


def layout(q, dt, nch, batch_cpw=0):
    """(chunks per group, groups) of pass 2 for a field of nch chunks."""
    if batch_cpw:
        per_tile, at_least, totals = 4 * batch_cpw, 64, False
    else:
        per_tile = 8 if dt == np.float32 and q != "abs" else 4
        at_least, totals = 16, -(-nch // per_tile) <= 4096
    tiles = -(-nch // per_tile)
    tpg = max(-(-at_least // per_tile), -(-tiles // 1024))
    if totals:
        tpg = -(-tpg // 4) * 4
    return tpg * per_tile, -(-tiles // tpg)


def hard_field(dt, cpg, ngroups, seed):
    """A smooth field of ngroups whole groups of cpg chunks (the last chunk 24
    values short) with hot groups 1, ngroups // 2 and the last, and a group
    of mixed rows that is not hot."""
    rng = np.random.default_rng(seed)
    cap = CAP[dt]
    n = cpg * ngroups * CHUNK - 24
    x = np.resize(synth.sines_1d(1 << 18, seed, dtype=dt), n)

    def rows(g, counts):
        for i, k in enumerate(counts):
            c = (g * cpg + i) * CHUNK
            v = x[c: c + CHUNK]
            v[:] = 0.5
            v[rng.permutation(v.size)[: min(k, v.size)]] = np.nan

    mixed = [31, 32, 33, 1, 0, 64, cap, cap + 1]
    for g in (1, ngroups // 2, ngroups - 1):
        rows(g, mixed + [CHUNK] * 8)
    rows(ngroups // 3, mixed)
    if cpg > 16:  # the ragged chunk is far from the rows above
        x[-(CHUNK - 24):] = np.nan
    return x


def check_input(st, dt, n, cpg, ngroups):
    """The groups are hot, or not, and hold what they should, by the stream's
    chunk table."""
    cap = CAP[dt]
    nch = -(-n // CHUNK)
    assert nch == cpg * ngroups
    k = int(st[16:24].view(np.uint64)[0])
    at = (64 + 4 * n + 15) // 16 * 16
    table = np.append(st[at: at + 8 * nch].view(np.uint64).astype(np.int64), k)
    cnt = np.diff(table).reshape(ngroups, cpg)
    own = cnt.sum(axis=1)
    hot = np.flatnonzero((own > 1024) & ((own - 1024) * ngroups > 4 * k))
    assert list(hot) == [1, ngroups // 2, ngroups - 1], hot
    for g in hot:
        assert {31, 32, 33, 1, 0, 64, cap, cap + 1} <= set(cnt[g]), cnt[g]
    assert cnt[-1, -1] == CHUNK - 24
    cold = cnt[ngroups // 3]
    assert {31, 32, 33, cap, cap + 1} <= set(cold), cold


# groups of 16 and 32 chunks with totals; just past 4096 first-pass workgroups,
# groups of 20 and 40 chunks with group sums
ALONE = [("abs", np.float32, 150), ("rel", np.float32, 150), ("noa", np.float32, 150),
         ("abs", np.float64, 150), ("rel", np.float64, 150), ("noa", np.float64, 150),
         ("abs", np.float32, 820), ("rel", np.float32, 820), ("abs", np.float64, 820)]


def alone(q, dt, ngroups):
    waves = 8 if dt == np.float32 and q != "abs" else 4
    tiles = ngroups * 5 if ngroups > 800 else ngroups * 4
    cpg, ng = layout(q, dt, tiles * waves)
    assert ng == ngroups and (tiles <= 4096) == (ngroups < 800)
    x = hard_field(dt, cpg, ng, 31)
    st = O.quantize_mt(q, x, EB)
    check_input(st, dt, x.size, cpg, ng)
    return x, st


@pytest.mark.parametrize("q,dt,ngroups", [a for a in ALONE if a[2] < 800])
def test_inputs(q, dt, ngroups):
    alone(q, dt, ngroups)


@pytest.mark.gpu
@pytest.mark.parametrize("q,dt,ngroups", ALONE)
def test_hot_groups(q, dt, ngroups):
    import torch
    import paper_2407_15037_amd as lcq
    x, want = alone(q, dt, ngroups)
    xt = torch.from_numpy(x).cuda()
    ws = torch.full((lcq.workspace_bytes(q, xt.dtype, x.size),), 0xA5, dtype=torch.uint8,
                    device="cuda")
    out = torch.full((lcq.max_stream_bytes(xt.dtype, x.size),), 0x5A, dtype=torch.uint8,
                     device="cuda")
    announce("hot groups", q, np.dtype(dt).name, x.size)
    buf, nb = lcq.quantize(xt, q, EB, out=out, ws=ws)
    assert first_diff(buf[: int(nb.item())].cpu().numpy(), want) is None


def dense_field(dt, nch, seed):
    """Every chunk with 60 to cap + 20 outliers: groups move more than one
    window of staged rows, none is hot, some chunks are over the cap."""
    rng = np.random.default_rng(seed)
    x = np.full(nch * CHUNK - 24, 0.5, dt)
    for c, k in enumerate(rng.integers(60, CAP[dt] + 21, nch)):
        v = x[c * CHUNK: (c + 1) * CHUNK]
        v[rng.permutation(v.size)[:k]] = np.nan
    return x


@pytest.mark.gpu
@pytest.mark.parametrize("dt", [np.float32, np.float64])
@pytest.mark.parametrize("q", ["abs", "rel"])
@pytest.mark.parametrize("nch", [33, 47, 64, 700])
def test_dense_everywhere(q, dt, nch):
    import torch
    import paper_2407_15037_amd as lcq
    from paper_2407_15037_amd.batch import BatchPlan
    x = dense_field(dt, nch, nch)
    want = O.quantize(q, x, EB)
    xt = torch.from_numpy(x).cuda()
    announce("dense everywhere", q, np.dtype(dt).name, x.size)
    buf, nb = lcq.quantize(xt, q, EB)
    assert first_diff(buf[: int(nb.item())].cpu().numpy(), want) is None
    plan = BatchPlan([{"x": xt, "q": q, "eb": EB}])
    plan.quantize()
    f = plan.fields[0]
    assert first_diff(f["stream"][: int(f["nbytes"].item())].cpu().numpy(), want) is None


@pytest.mark.gpu
@pytest.mark.parametrize("cpw", [1, 4])
def test_hot_groups_in_a_batch(cpw):
    import torch
    from paper_2407_15037_amd.batch import BatchPlan
    fields, want = [], []
    for q, dt in (("abs", np.float32), ("rel", np.float32), ("noa", np.float64)):
        cpg, ng = layout(q, dt, 64 * 100, cpw)
        assert (cpg, ng) == (64, 100)
        x = hard_field(dt, cpg, ng, 33)
        st = O.quantize_mt(q, x, EB)
        check_input(st, dt, x.size, cpg, ng)
        fields.append({"x": torch.from_numpy(x).cuda(), "q": q, "eb": EB})
        want.append(st)
    announce("hot groups in a batch", cpw)
    plan = BatchPlan(fields, tune=f"batch=0 f32={cpw} f64={cpw}")
    plan.quantize()
    for f, st in zip(plan.fields, want):
        got = f["stream"][: int(f["nbytes"].item())].cpu().numpy()
        assert first_diff(got, st) is None


@pytest.mark.gpu
@pytest.mark.parametrize("dt", [np.float32, np.float64])
def test_groups_of_several_batches(dt):
    """Groups of 300 chunks (307,200 in all): a pass-2 workgroup takes 256 of
    them, then 44, with 0 to 60 outliers in most, a few over the stage cap and
    one hot group of short, full and over-cap rows.  Codes, chunk table and
    outliers follow from the input: every value is either 0.5 or a NaN with its
    own payload."""
    import torch
    import paper_2407_15037_amd as lcq
    from paper_2407_15037_amd.batch import BatchPlan
    nch, cap = 300 * 1024, CAP[dt]
    assert layout("abs", dt, nch) == (300, 1024)
    g = torch.Generator().manual_seed(9)
    cnt = torch.randint(0, 61, (nch,), generator=g)
    over = torch.rand(nch, generator=g) < 0.01
    cnt[over] = torch.randint(cap + 1, 400, (int(over.sum()),), generator=g)
    cnt[600 * 300: 601 * 300] = torch.tensor([20, cap, CHUNK] * 100)
    cnt[-1] = CHUNK
    own = cnt.reshape(1024, 300).sum(1)
    assert int(own[600]) > 1024 + 4 * int(own.sum()) // 1024 and int(own[:256].max()) > 2048
    cnt = cnt.cuda()
    idt, tdt = ((torch.int32, torch.float32) if dt == np.float32 else (torch.int64, torch.float64))
    n = nch * CHUNK
    pos = torch.arange(CHUNK, device="cuda")
    x = torch.full((nch, CHUNK), 0.5, dtype=tdt, device="cuda")
    want = []
    for c0 in range(0, nch, 1 << 14):  # (slices, to keep the index tensors small)
        c = torch.arange(c0, min(c0 + (1 << 14), nch), device="cuda")
        mask = (pos[None] * 389 + c[:, None] * 17) % CHUNK < cnt[c][:, None]
        word = (c[:, None] * CHUNK + pos[None]) & 0x3FFFFF
        word |= 0x7FC00000 if dt == np.float32 else 0x7FF8000000000000
        sl = x[c0: c0 + c.numel()].view(idt)
        sl[mask] = word.to(idt)[mask]
        want.append(sl[mask])
    want, x = torch.cat(want), x.reshape(-1)
    table = torch.cumsum(cnt, 0) - cnt
    k = int(cnt.sum())
    ct = (64 + 4 * n + 15) // 16 * 16
    oo = (ct + 8 * nch + 15) // 16 * 16

    def check(buf, nb):
        size = int(nb.item())
        assert size == oo + k * x.element_size()
        assert int(buf[16:24].view(torch.int64).item()) == k
        assert torch.equal(buf[ct: ct + 8 * nch].view(torch.int64), table)
        assert torch.equal(buf[oo: size].view(idt), want)
        codes = buf[64: 64 + 4 * n].view(torch.int32).reshape(nch, CHUNK)
        assert torch.equal((codes == -(1 << 31)).sum(1), cnt)
        assert int(torch.unique(codes[codes != -(1 << 31)]).numel()) == 1

    announce("groups of several batches", np.dtype(dt).name)
    check(*lcq.quantize(x, "abs", EB))
    plan = BatchPlan([{"x": x, "q": "abs", "eb": EB}])
    plan.quantize()
    check(plan.fields[0]["stream"], plan.fields[0]["nbytes"])
