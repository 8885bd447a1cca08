"""Steps whose terms are grouped as records: the borders of the dispatch, one and few rows, buckets of more records than a workgroup
takes, long rows in both tables, every or no centre its own run, the optimizers' marks of the rows of a batch and the one-table step."""
import numpy as np
import pytest
import torch

from tolerances import EMB_ATOL, LOSS_RTOL, assert_emb_close, assert_half_close

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _dev(a):
    return torch.as_tensor(np.ascontiguousarray(a)).to(DEV)


def _batch(kind, n, b, k, rng):
    c = np.repeat(rng.integers(0, n, b // 5 + 1), 5)[:b].astype(np.int32)
    o, neg = rng.integers(0, n, b).astype(np.int32), rng.integers(0, n, (b, k)).astype(np.int32)
    if kind == "hub":                       # half of all terms and of all runs in one row
        o[rng.random(b) < 0.5] = n - 1
        neg[rng.random((b, k)) < 0.5] = n - 1
        c[(np.arange(b) // 5) % 2 == 0] = n // 2
    elif kind == "runs of one":
        c = rng.permutation(np.arange(b) % n).astype(np.int32)
    elif kind == "one run":
        c[:] = n // 3
    return c, o, neg


def _tables(n, dim, count, seed, scale=0.3):
    g = torch.Generator().manual_seed(seed)
    return [(torch.rand((n, dim), generator=g) - 0.5) * scale for _ in range(count)]


# terms: 5 * 2^16 and one less on 2^16 rows, 5 * 2^17 on one row more; 1 to 32 rows; up to 256, 1024 and 2048 buckets; tiles of 2048,
# 4096 and 8192 records; a row per bucket with more records than a workgroup takes
@pytest.mark.parametrize("kind,n,b,k", [
    ("even", 65_536, 54_614, 5), ("even", 65_536, 54_613, 5), ("even", 65_537, 109_227, 5), ("even", 65_537, 109_226, 5),
    ("even", 1, 65_536, 4), ("even", 2, 70_001, 4), ("even", 33, 70_001, 4), ("even", 5_000, 350_003, 0), ("hub", 20_000, 120_000, 5),
    ("hub", 300_000, 262_145, 5), ("runs of one", 70_000, 400_000, 1), ("one run", 70_000, 131_073, 7), ("hub", 3_000_001, 699_051, 6),
    ("even", (1 << 24) - 5, 131_101, 4)])
@pytest.mark.parametrize("fmt", ["f32", "bf16"])
def test_step(oracle, kind, n, b, k, fmt):
    from paper_2407_15452_amd import binding as gs
    dim = 8 if n > 1_000_000 else 24
    c, o, neg = _batch(kind, n, b, k, np.random.default_rng(n + b))
    tabs = [t.to(torch.float32 if fmt == "f32" else torch.bfloat16) for t in _tables(n, dim, 2, n)]
    host = [t.numpy().copy() if fmt == "f32" else t.view(torch.int16).numpy().view(np.uint16).copy() for t in tabs]
    dev = [t.to(DEV) for t in tabs]
    lr = 1e-5 if n < 100 else 1e-4          # (rows of 10^5 terms)
    want = oracle.sgns_step(*host, c, o, neg, lr, dtype=oracle.F32 if fmt == "f32" else oracle.BF16)
    loss = gs.gs_sgns_step(*dev, _dev(c), _dev(o), _dev(neg), lr)
    assert abs(float(loss.item()) - want) <= LOSS_RTOL * abs(want)
    for d, h in zip(dev, host):
        if fmt == "f32":
            assert_emb_close(d.cpu().numpy(), h)
        else:                               # (tables of a few rows: one element that rounds the other way is more than the share)
            assert_half_close(d.view(torch.int16).cpu().numpy().view(np.uint16), h, fmt,
                              flip_fraction=None if h.size > 20_000 else 2.0 / h.size)


@pytest.mark.parametrize("b,k,mean", [(100_000, 4, 64), (1_400_000, 0, 256), (300_000, 3, 256)])
@pytest.mark.parametrize("less", [0, 256])
def test_rows_of_whole_segments(oracle, b, k, mean, less):
    """Rows of a few records more and less than one, two and seventeen segments of 64 or 256, in both tables, so that further segments start
    everywhere; also as the sorted records (or counters) that a little less room leaves."""
    from paper_2407_15452_amd import binding as gs
    rng = np.random.default_rng(b)

    def ids(count):
        sizes = rng.choice([1, mean - 1, mean, mean + 1, 2 * mean, 2 * mean + 1, 17 * mean + 3], count // mean + 200, p=[.3, .1, .2, .2, .1, .05, .05])
        rows = np.repeat(rng.permutation(sizes.size), sizes)[:count]
        assert rows.size == count
        return rows.astype(np.int32), sizes.size

    terms, n_out = ids(b * (k + 1))
    terms = rng.permutation(terms).reshape(b, k + 1)
    c, n_in = ids(b)
    c = rng.permutation(c)                  # (nearly every centre its own run)
    n, dim, lr = max(n_out, n_in), 8, 1e-4
    o, neg = np.ascontiguousarray(terms[:, 0]), np.ascontiguousarray(terms[:, 1:])
    tabs = _tables(n, dim, 2, n)
    host, dev = [t.numpy().copy() for t in tabs], [t.to(DEV) for t in tabs]
    want = oracle.sgns_step(*host, c, o, neg, lr)
    ws = torch.empty(gs.gs_sgns_step_workspace_bytes(b, n, k, dim, gs.GS_F32) - less, dtype=torch.uint8, device=DEV)
    loss = gs.gs_sgns_step(*dev, _dev(c), _dev(o), _dev(neg), lr, ws=ws)
    assert abs(float(loss.item()) - want) <= LOSS_RTOL * abs(want)
    for d, h in zip(dev, host):
        assert_emb_close(d.cpu().numpy(), h)


@pytest.mark.parametrize("n,b,k", [(700, 1_500_000, 5), (5_000, 6_000_000, 5), (3_000_000, 5_800_000, 5), (9_000_000, 5_600_000, 5)])
def test_more_records_than_buckets_hold(n, b, k):
    """Tiles of 16,384 records and few buckets, and every bucket split (or, of more than 2^23 rows, sorted records): bit for bit what sorted
    records and counters in less room give (the sums are exact, and chunks of a forward group the same)."""
    from paper_2407_15452_amd import binding as gs
    gen = torch.Generator(device=DEV).manual_seed(n)
    ids = [(torch.rand(m, generator=gen, device=DEV) ** 2 * n).to(torch.int32).clamp_(0, n - 1) for m in (b // 4, b, b * k)]
    c, o, neg = ids[0].repeat_interleave(4), ids[1], ids[2].view(b, k)
    assert c.numel() == b
    tabs = [t.to(DEV) for t in _tables(n, 4, 2, n)]
    size = gs.gs_sgns_step_workspace_bytes(b, n, k, 4, gs.GS_F32)
    ws = torch.empty(size, dtype=torch.uint8, device=DEV)
    results = []
    for room in (size, size - 256, size // 256 * 256 * 3 // 4):
        mine = [t.clone() for t in tabs]
        try:
            loss = gs.gs_sgns_step(*mine, c, o, neg, 1e-7, ws=ws[:room])
        except gs.GsError as e:
            assert e.status == gs.GS_EWORKSPACE and room < size - 256
            continue
        results.append((loss, *mine))
    assert all(torch.equal(x, y) for r in results[1:] for x, y in zip(r, results[0])) and np.isfinite(float(results[0][0].item()))


@pytest.mark.parametrize("kind,n,b,k", [("even", 65_536, 54_614, 5), ("hub", 40_000, 60_000, 5), ("hub", 700_000, 110_000, 5)])
@pytest.mark.parametrize("call", ["momentum", "adam", "line1"])
def test_optimizers_and_one_table(oracle, call, kind, n, b, k):
    from paper_2407_15452_amd import binding as gs
    dim, lr = 12, 1e-3
    c, o, neg = _batch(kind, n, b, k, np.random.default_rng(n))
    tabs = _tables(n, dim, 4, n)
    if call == "line1":
        tabs = tabs[:1]
    elif call == "adam":
        tabs += [t.abs() + 0.01 for t in _tables(n, dim, 2, n + 1, 0.1)]          # (denominators well above zero)
    host, dev = [t.numpy().copy() for t in tabs], [t.to(DEV) for t in tabs]
    ids = (_dev(c), _dev(o), _dev(neg))
    if call == "momentum":
        want, loss = oracle.sgns_momentum_step(*host, c, o, neg, lr, 0.875), gs.gs_sgns_momentum_step(*dev, *ids, lr, 0.875)
    elif call == "adam":
        rates = (lr, 0.9, 0.999, 1e-8, 5)
        want, loss = oracle.sgns_adam_step(*host, c, o, neg, *rates), gs.gs_sgns_adam_step(*dev, *ids, *rates)
    else:
        want, loss = oracle.line1_step(*host, c, o, neg, lr), gs.gs_line1_step(*dev, *ids, lr)
    assert abs(float(loss.item()) - want) <= LOSS_RTOL * abs(want)
    for i, (d, h) in enumerate(zip(dev, host)):
        got = d.cpu().numpy()
        if call == "adam" and i < 2:
            assert np.abs(got - h).max() <= EMB_ATOL
        elif call == "adam":
            assert (np.abs(got - h) <= 1e-6 + 1e-5 * np.abs(h)).all()
        else:
            assert_emb_close(got, h)


@pytest.mark.parametrize("fmt", ["bf16", "f16"])
@pytest.mark.parametrize("call,n,b,k,dim", [("momentum", 40_000, 60_000, 5, 24), ("momentum", 40_000, 60_000, 5, 136), ("momentum", 300_000, 110_000, 5, 264),
                                            ("line1", 40_000, 60_000, 5, 24), ("line1", 300_000, 110_000, 5, 264)])
def test_16bit_momentum_and_one_table(oracle, call, fmt, n, b, k, dim):
    from paper_2407_15452_amd import binding as gs
    dtype, code, lr = torch.bfloat16 if fmt == "bf16" else torch.float16, oracle.BF16 if fmt == "bf16" else oracle.F16, 5e-3
    c, o, neg = _batch("hub", n, b, k, np.random.default_rng(dim))
    tabs = [t.to(dtype) for t in _tables(n, dim, 4 if call == "momentum" else 1, dim)]
    host = [t.view(torch.int16).numpy().view(np.uint16).copy() for t in tabs]
    dev, ids = [t.to(DEV) for t in tabs], (_dev(c), _dev(o), _dev(neg))
    if call == "momentum":
        want, loss = oracle.sgns_momentum_step(*host, c, o, neg, lr, 0.875, dtype=code), gs.gs_sgns_momentum_step(*dev, *ids, lr, 0.875)
    else:
        want, loss = oracle.line1_step(*host, c, o, neg, lr, dtype=code), gs.gs_line1_step(*dev, *ids, lr)
    assert abs(float(loss.item()) - want) <= LOSS_RTOL * abs(want)
    for d, h in zip(dev, host):             # (one table: a row is rounded with its context terms, then with its source terms)
        assert_half_close(d.view(torch.int16).cpu().numpy().view(np.uint16), h, fmt, steps=2 if call == "line1" else 1)


def test_bad_ids_and_products_out_of_range():
    """Both turn the loss into NaN; the ids are read as row 0."""
    from paper_2407_15452_amd import binding as gs
    n, b, k = 60_000, 60_000, 5
    c, o, neg = _batch("even", n, b, k, np.random.default_rng(1))
    for ids, lr in (((c, o, np.where(neg == neg[7, 2], n, neg)), 1e-3), ((np.where(c == c[5], -1, c), o, neg), 1e-3), ((c, o, neg), 1e6)):
        dev = [t.to(DEV) for t in _tables(n, 8, 2, 3)]
        assert np.isnan(float(gs.gs_sgns_step(*dev, *(_dev(x.astype(np.int32)) for x in ids), lr).item()))


@pytest.mark.parametrize("fmt", ["bf16", "f16"])
@pytest.mark.parametrize("dim", [8, 120, 136, 248, 264, 504, 520, 1016])
@pytest.mark.parametrize("n,b,k", [(100_000, 1_500, 6), (20_000, 9_000, 3), (30_000, 30_000, 10)])
def test_short_16bit_rows(oracle, fmt, dim, n, b, k):
    """Rows that leave lanes of the forward kernel without a piece, and terms that do not fill its blocks of rows: two launches (or, of
    wide rows, counters over the keys of the batch), counters, grouped records."""
    from paper_2407_15452_amd import binding as gs
    dtype = torch.bfloat16 if fmt == "bf16" else torch.float16
    c, o, neg = _batch("even", n, b, k, np.random.default_rng(dim))
    tabs = [t.to(dtype) for t in _tables(n, dim, 2, dim)]
    host = [t.view(torch.int16).numpy().view(np.uint16).copy() for t in tabs]
    dev = [t.to(DEV) for t in tabs]
    want = oracle.sgns_step(*host, c, o, neg, 0.01, dtype=oracle.BF16 if fmt == "bf16" else oracle.F16)
    loss = gs.gs_sgns_step(*dev, _dev(c), _dev(o), _dev(neg), 0.01)
    assert abs(float(loss.item()) - want) <= LOSS_RTOL * abs(want)
    for d, h in zip(dev, host):
        assert_half_close(d.view(torch.int16).cpu().numpy().view(np.uint16), h, fmt)


@pytest.mark.parametrize("fmt", ["bf16", "f16"])
@pytest.mark.parametrize("dim", [136, 256, 264, 512])
@pytest.mark.parametrize("n,b,k", [(100_000, 1_500, 1), (30_000, 30_000, 1), (30_000, 180_001, 1), (30_000, 330_001, 0)])
def test_16bit_rows_with_one_negative_or_none(oracle, fmt, dim, n, b, k):
    """Blocks of two rows: two launches, counters, grouped records."""
    test_short_16bit_rows(oracle, fmt, dim, n, b, k)


@pytest.mark.parametrize("fmt", ["bf16", "f16"])
@pytest.mark.parametrize("table", [0, 1])
@pytest.mark.parametrize("n,b,k", [(100_000, 1_500, 6), (20_000, 9_000, 3), (30_000, 30_000, 10)])
def test_infinity_in_the_last_piece(fmt, table, n, b, k):
    """An infinity among the last columns of a row that leaves lanes of the forward kernel without a piece: the rows come out as
    the same rows do with zeros up to the columns that fill the lanes."""
    from paper_2407_15452_amd import binding as gs
    dtype = torch.bfloat16 if fmt == "bf16" else torch.float16
    c, o, neg = (_dev(x) for x in _batch("even", n, b, k, np.random.default_rng(b)))
    wide = [torch.zeros((n, 256), dtype=dtype) for _ in range(2)]
    for w, t in zip(wide, _tables(n, 200, 2, n)):
        w[:, :200] = t.to(dtype)
    wide[table][(c if table == 0 else o)[17].item(), 197] = float("inf")
    short = [w[:, :200].contiguous().to(DEV) for w in wide]
    wide = [w.to(DEV) for w in wide]
    for tabs in (short, wide):
        assert np.isnan(float(gs.gs_sgns_step(*tabs, c, o, neg, 0.01).item()))
    for s, w in zip(short, wide):
        # (NaN may carry any bits)
        s, w = s.cpu(), w[:, :200].cpu()
        assert torch.equal(s.isnan(), w.isnan())
        assert torch.equal(s.nan_to_num(nan=0.0), w.nan_to_num(nan=0.0))
