"""The step on sorted records (batches of at least 9 * 2^19 terms, 2^20 or, with at most one negative, 2^21 on at
most 2^16 rows) and just below, against the CPU reference: a handful of rows with everything in them, rows around the segment length (256 terms) and around slice borders,
rows of a few terms on a large table, both table types and the one-table step."""
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
