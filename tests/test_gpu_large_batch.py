"""Large steps against the CPU reference.  Up to 2^24 rows their terms are records that are grouped by row (test_gpu_grouping.py has that way's
borders): a handful of rows with everything in them, rows around the segment length (256 terms) and around slice borders, rows of a few terms on a
large table, both table types and the one-table step.  On more rows the records are sorted (at least 9 * 2^19 terms): rows of whole segments and
long ones, every width of rows, both tables or one, negatives drawn and pairs made in the call."""
import numpy as np
import pytest
import torch

from tolerances import LOSS_RTOL, assert_emb_close, assert_half_close

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _dev(a):
    return torch.as_tensor(np.ascontiguousarray(a)).to(DEV)


def _ids(kind, n, count, rng):
    if kind == "few":
        return rng.integers(0, min(n, 5), count).astype(np.int32)
    if kind == "segments":                 # row r has 250 + r % 14 terms: just below, at and above one segment
        rows = np.repeat(np.arange(n), 250 + np.arange(n) % 14)[:count]
        assert rows.size == count
        return rng.permutation(rows).astype(np.int32)
    return rng.integers(0, n, count).astype(np.int32)


@pytest.mark.parametrize("kind,n,k,b", [("few", 7, 3, 1 << 18), ("few", 1, 3, 1 << 18),
                                        ("even", 3_000, 1, (1 << 20) - 1), ("even", 3_000, 1, 1 << 20),
                                        ("even", 65_536, 5, 174_762), ("even", 65_536, 5, 174_763),
                                        ("even", 65_537, 5, 174_763),
                                        ("few", 7, 3, 1 << 20), ("segments", 18_000, 0, (1 << 22) + 1),
                                        ("even", 3_000, 5, 699_051), ("even", 700_000, 2, 1_572_864),
                                        ("even", 20_000_000, 6, 674_085)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_step(oracle, kind, n, k, b, dtype):
    from paper_2407_15452_amd import binding as gs
    dim = 8
    rng = np.random.default_rng(n)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator().manual_seed(n)
    tabs = [((torch.rand((n, dim), generator=gen) - 0.5) * 0.6).to(tdt) for _ in range(2)]
    host = [t.numpy().copy() if dtype == "f32" else t.view(torch.int16).numpy().view(np.uint16).copy() for t in tabs]
    dev = [t.to(DEV) for t in tabs]
    c = np.repeat(rng.integers(0, n, b // 5 + 1), 5)[:b].astype(np.int32)
    o = _ids(kind, n, b, rng)
    neg = _ids("even" if kind == "segments" else kind, n, b * k, rng).reshape(b, k)
    lr = 1e-4 if n < 5_000 else 0.01       # (rows of 10^5 terms)
    want = oracle.sgns_step(*host, c, o, neg, lr, dtype=oracle.F32 if dtype == "f32" else oracle.BF16)
    loss = gs.gs_sgns_step(*dev, _dev(c), _dev(o), _dev(neg), lr)
    assert abs(float(loss.item()) - want) <= LOSS_RTOL * abs(want)
    for d, h in zip(dev, host):
        if dtype == "f32":
            assert_emb_close(d.cpu().numpy(), h)
        else:
            # (tables of a few rows: one element that rounds the other way is more than the share)
            assert_half_close(d.view(torch.int16).cpu().numpy().view(np.uint16), h, dtype,
                              flip_fraction=None if n > 1000 else 2.0 / h.size)


def test_one_table(oracle):
    from paper_2407_15452_amd import binding as gs, inputs
    n, dim, k, b = 4_000, 12, 4, 838_861
    rng = np.random.default_rng(1)
    w = inputs.random_tables(n, dim, 8, 0.3)[0]
    h, d = w.numpy().copy(), w.to(DEV)
    src, dst = rng.integers(0, n, b).astype(np.int32), rng.integers(0, n, b).astype(np.int32)
    neg = rng.integers(0, n, (b, k)).astype(np.int32)
    want = oracle.line1_step(h, src, dst, neg, 1e-3)
    loss = gs.gs_line1_step(d, _dev(src), _dev(dst), _dev(neg), 1e-3)
    assert abs(float(loss.item()) - want) <= LOSS_RTOL * abs(want)
    assert_emb_close(d.cpu().numpy(), h)


def test_reports_bad_ids_and_repeats_the_bits():
    """An id that is not a row turns the loss into NaN; the same batch twice gives the same bits.  (Workspaces
    without room for the records: test_gpu_step_routes.py.)"""
    from paper_2407_15452_amd import binding as gs, inputs
    n, dim, k, b = 2_000, 8, 5, 699_051
    rng = np.random.default_rng(2)
    w_in, w_out = inputs.random_tables(n, dim, 3, 0.3)
    c, o = rng.integers(0, n, b).astype(np.int32), rng.integers(0, n, b).astype(np.int32)
    neg = rng.integers(0, n, (b, k)).astype(np.int32)
    runs = []
    for _ in range(2):
        d = [w_in.to(DEV), w_out.to(DEV)]
        gs.gs_sgns_step(*d, _dev(c), _dev(o), _dev(neg), 1e-3)
        runs.append(d)
    assert torch.equal(runs[0][0], runs[1][0]) and torch.equal(runs[0][1], runs[1][1])
    neg[b // 2, 1] = n
    assert np.isnan(float(gs.gs_sgns_step(*runs[0], _dev(c), _dev(o), _dev(neg), 1e-3).item()))


SORTED_ROWS = (1 << 24) + 1                 # the fewest that are not grouped


def _whole_segments(rows, count, rng):
    """Ids in any order, of which each has up to three terms, or up to two more or less than one, two or seventeen segments of 256."""
    sizes = rng.choice([1, 2, 3, 254, 255, 256, 257, 258, 511, 512, 513, 4352, 4355], count // 100 + 200,
                       p=[.3, .2, .1, .04, .06, .06, .06, .04, .03, .04, .03, .02, .02])
    ids = np.repeat(rng.permutation(rows[:sizes.size]), sizes)[:count]
    assert sizes.size <= rows.size and ids.size == count
    return rng.permutation(ids).astype(np.int32)


@pytest.mark.parametrize("call,fmt,dim", [("step", "f32", 4), ("step", "f32", 132), ("step", "f16", 264), ("step", "bf16", 520), ("step", "f32", 516),
                                          ("line1", "f32", 8), ("line1", "bf16", 264)])
def test_sorted_records(oracle, call, fmt, dim):
    """Rows of up to 256, 1024, 2048 and 4096 bytes.  The reference's tables hold the rows that the batch names; all others
    have to come out as they went in."""
    from paper_2407_15452_amd import binding as gs
    n, k, b = SORTED_ROWS, 5, 786_433
    rng = np.random.default_rng(dim)
    named = np.unique(np.concatenate([[0, n - 1], rng.integers(0, n, 60_000)]))
    rows = rng.permutation(named.size)                     # rows of the reference's tables
    terms = _whole_segments(rows, b * (k + 1), rng).reshape(b, k + 1)
    o, neg = np.ascontiguousarray(terms[:, 0]), np.ascontiguousarray(terms[:, 1:])
    c = np.repeat(_whole_segments(rows, b // 3 + 1, rng), 3)[:b]
    tdt = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[fmt]

    def table(seed):
        return torch.rand((n, dim), generator=torch.Generator(device=DEV).manual_seed(seed), device=DEV).sub_(0.5).mul_(0.6).to(tdt)

    tabs = [table(i) for i in range(1 if call == "line1" else 2)]
    at = _dev(named)
    host = [t[at].cpu().numpy() if fmt == "f32" else t[at].view(torch.int16).cpu().numpy().view(np.uint16) for t in tabs]
    ids = [_dev(named[x].astype(np.int32)) for x in (c, o, neg)]
    lr, code = 0.02, {"f32": oracle.F32, "bf16": oracle.BF16, "f16": oracle.F16}[fmt]
    if call == "line1":
        want, loss = oracle.line1_step(*host, c, o, neg, lr, dtype=code), gs.gs_line1_step(*tabs, *ids, lr)
    else:
        want, loss = oracle.sgns_step(*host, c, o, neg, lr, dtype=code), gs.gs_sgns_step(*tabs, *ids, lr)
    assert abs(float(loss.item()) - want) <= LOSS_RTOL * abs(want)
    for i, (t, h) in enumerate(zip(tabs, host)):
        got = t[at].cpu()
        if fmt == "f32":
            assert_emb_close(got.numpy(), h)
        else:               # (one table: a row is rounded with its context terms, then with its source terms)
            assert_half_close(got.view(torch.int16).numpy().view(np.uint16), h, fmt, steps=2 if call == "line1" else 1)
        as_before = table(i)
        as_before[at] = t[at]
        assert torch.equal(t, as_before)


@pytest.mark.parametrize("call", ["fused", "from_walks"])
def test_sorted_records_of_pairs_made_in_the_call(call):
    """Negatives drawn and pairs made in the call: the bits of the step on the same ones made before it."""
    from paper_2407_15452_amd import binding as gs
    n, k, dim, length, window, first = SORTED_ROWS, 7, 8, 20, 5, 3
    gen = torch.Generator(device=DEV).manual_seed(1)
    walks = (torch.rand((4_000, length), generator=gen, device=DEV) ** 4 * n).to(torch.int32).clamp_(0, n - 1)
    walks[::7, 13:] = -1
    noise = gs.gs_alias_build(torch.tensor([0, n], dtype=torch.int64, device=DEV), torch.rand(n, generator=gen, device=DEV) ** 8)
    c, o, pairs = gs.gs_make_pairs(walks, window)
    b = ((9 << 19) + k) // (k + 1) + 1
    assert pairs >= first + b
    c, o = c[first:first + b].clone(), o[first:first + b].clone()
    tabs = [torch.rand((n, dim), generator=gen, device=DEV).sub_(0.5) for _ in range(2)]
    mine = [t.clone() for t in tabs]
    loss = gs.gs_sgns_step(*tabs, c, o, gs.gs_sample_negatives(noise, n, b, k, 9, pair_index_base=77), 0.01)
    if call == "fused":
        own = gs.gs_sgns_step_fused(*mine, c, o, noise, k, 9, 0.01, pair_index_base=77)
    else:
        own = gs.gs_sgns_step_from_walks(*mine, walks, window, gs.gs_pair_offsets(walks, window), first, b, noise, k, 9, 0.01, pair_index_base=77)
    assert float(own.item()) == float(loss.item()) and np.isfinite(float(loss.item()))
    assert all(torch.equal(x, y) for x, y in zip(mine, tabs))
