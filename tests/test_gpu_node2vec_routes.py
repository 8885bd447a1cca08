"""The node2vec walker against the CPU reference, bit for bit, on graphs that put its reads at both ends of the arrays: 4095 to 2^23
entries, two and three nodes, dead ends, rows of equal length, 31 to 131,073 walks from the last rows on, uniform and weighted draws
(all of them launches of teams of lanes); and its state machine, a lane per walk, which takes more than 163,840 unweighted walks of many
attempts: walks that end inside a window of 16 positions and behind several, rows whose bounds are the last 16 bytes, dead
ends before and after a window has been written out."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
ENTRIES = 1 << 22


def _dev(a):
    return torch.as_tensor(np.ascontiguousarray(a)).to(DEV)


def _graph(kind, n, entries):
    rng = np.random.default_rng(n)
    if kind == "dead-ends":               # half of the nodes have no row
        return rng.integers(0, n // 2, entries).astype(np.int32) * 2, rng.integers(0, n, entries).astype(np.int32)
    return rng.integers(0, n, entries).astype(np.int32), rng.integers(0, n, entries).astype(np.int32)


@pytest.mark.parametrize("kind,n,entries,walks", [("even", 3, ENTRIES, 512), ("even", 2, ENTRIES + 1, 512),
                                                  ("even", 60, 4096, 32), ("even", 60, 4095, 33), ("even", 60, 4097, 31),
                                                  ("even", 5000, ENTRIES, 575), ("even", 5000, ENTRIES - 1, 575),
                                                  ("even", 5000, ENTRIES + 3, 511), ("even", 5000, 3 << 19, 1 << 14), ("even", 5000, 3 << 18, 512),
                                                  ("dead-ends", 300_000, ENTRIES + 2, 131_072),
                                                  ("dead-ends", 300_000, ENTRIES + 2, 131_073),
                                                  ("dead-ends", 500_000, ENTRIES, 5_000), ("rows", 4096, 1 << 23, 575)])
def test_same_walks(oracle, kind, n, entries, walks):
    from paper_2407_15452_amd import binding as gs
    w = np.random.default_rng(1).lognormal(0, 1, entries).astype(np.float32)
    if kind == "rows":                    # rows of equal length, as they are
        off = np.arange(n + 1, dtype=np.int32) * (entries // n)
        nb, ww = np.sort(np.random.default_rng(2).integers(0, n, (n, entries // n)).astype(np.int32), axis=1).ravel(), w
    else:
        off, nb, ww = oracle.csr_build(*_graph(kind, n, entries), w, n, 0)
    assert nb.size == entries
    table = oracle.alias_build(off, ww)
    starts = (n - 1 - np.arange(walks) % n).astype(np.int32)     # the last rows first
    length = 9 if walks > 100_000 else 24
    nbrs = _dev(nb)
    prob, alias = _dev(table[0]), _dev(table[1])
    packed = gs.gs_alias_pack(prob, alias)
    for p, q in ((0.5, 2.0), (2.0, 1.0), (4.0, 0.25), (1.0, 1.0)):
        for tab in (None, table):
            want = oracle.node2vec_walk(off, nb, starts, length, p, q, 5, alias=tab, walk_id_base=7)
            for dtype in (np.int32, np.int64):
                g = gs.Csr(_dev(off.astype(dtype)), nbrs)
                for a in ([None] if tab is None else [gs.Alias(prob, alias, packed), gs.Alias(prob, alias)]):
                    got = gs.gs_node2vec_walk(g, a, _dev(starts), length, p, q, 5, walk_id_base=7)
                    np.testing.assert_array_equal(got.cpu().numpy(), want)


@pytest.mark.parametrize("kind,n,entries,length", [("even", 3, 40_000, 33), ("dead-ends", 40_000, 300_000, 17),
                                                   ("dead-ends", 40_000, 300_000, 40), ("few-dead", 5000, 60_000, 40),
                                                   ("few-dead", 5000, 60_000, 33)])
def test_lane_per_walk(oracle, kind, n, entries, length):
    from paper_2407_15452_amd import binding as gs
    walks = 163_841
    if kind == "few-dead":                # one node in 40 has no row: most walks end behind their first window
        rng = np.random.default_rng(n)
        src = rng.integers(0, n, entries).astype(np.int32)
        dst = rng.integers(0, n, entries).astype(np.int32)
        src = np.where(src % 40 == 7, src - 1, src).astype(np.int32)
    else:
        src, dst = _graph(kind, n, entries)
    off, nb, _ = oracle.csr_build(src, dst, None, n, 0)
    starts = (n - 1 - np.arange(walks) % (n + 1)).astype(np.int32)       # the last rows first; -1, no node, among them
    want = oracle.node2vec_walk(off, nb, starts, length, 0.5, 2.0, 5, walk_id_base=7)
    if kind == "few-dead":                # walks that end in every window
        ends = (want >= 0).sum(1)
        assert all(((ends > lo) & (ends <= lo + 16) & (ends < length)).any() for lo in range(0, length - 1, 16))
    for dtype in (np.int32, np.int64):
        got = gs.gs_node2vec_walk(gs.Csr(_dev(off.astype(dtype)), _dev(nb)), None, _dev(starts), length, 0.5, 2.0, 5,
                                  walk_id_base=7)
        np.testing.assert_array_equal(got.cpu().numpy(), want)
