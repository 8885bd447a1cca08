"""The node2vec walker by teams of 1 to 64 lanes per walk and by a lane per walk, against the CPU reference, bit for bit: on
both sides of every number of walks at which the team changes, for settings that take many attempts, few and one, walks that
end in the middle of a window, dead ends, and graphs too small for a four-entry probe."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
MANY, FEW, ONE = (0.5, 2.0), (4.0, 0.25), (2.0, 1.0)      # p, q: about 4, 1 to 2 and 1 attempts a step


def _dev(a):
    return torch.as_tensor(np.ascontiguousarray(a)).to(DEV)


def _check(oracle, n, src, dst, walks, length, settings, ids=9):
    from paper_2407_15452_amd import binding as gs
    w = np.random.default_rng(3).lognormal(0, 1, src.size).astype(np.float32)
    off, nb, ww = oracle.csr_build(src, dst, w, n, 0)
    table = oracle.alias_build(off, ww)
    starts = (np.arange(walks) % (n + 1) - 1).astype(np.int32)           # -1, no node, among them
    prob, alias = _dev(table[0]), _dev(table[1])
    packed = gs.gs_alias_pack(prob, alias)
    for p, q in settings:
        for tab in (None, table):
            want = oracle.node2vec_walk(off, nb, starts, length, p, q, 11, alias=tab, walk_id_base=ids)
            for dtype in (np.int32, np.int64):
                g = gs.Csr(_dev(off.astype(dtype)), _dev(nb))
                for a in ([None] if tab is None else [gs.Alias(prob, alias, packed), gs.Alias(prob, alias)]):
                    got = gs.gs_node2vec_walk(g, a, _dev(starts), length, p, q, 11, walk_id_base=ids)
                    np.testing.assert_array_equal(got.cpu().numpy(), want)


def _graph(n, entries, dead):
    rng = np.random.default_rng(n)
    src = rng.integers(0, n // 2, entries) * 2 if dead else rng.integers(0, n, entries)
    return src.astype(np.int32), rng.integers(0, n, entries).astype(np.int32)


@pytest.mark.parametrize("walks,length", [(1, 40), (65, 33), (4096, 18), (4097, 18), (12_288, 17), (12_289, 17), (24_576, 9),
                                          (24_577, 9)])
def test_few_walks(oracle, walks, length):
    _check(oracle, 700, *_graph(700, 9000, False), walks, length, (MANY, FEW, ONE))


@pytest.mark.parametrize("walks,settings", [(49_152, (FEW, ONE)), (49_153, (FEW, ONE)), (163_840, (MANY,)), (163_841, (MANY,)),
                                            (1 << 18, (FEW,)), ((1 << 18) + 1, (FEW, (1.0, 1.0)))])
def test_many_walks(oracle, walks, settings):
    _check(oracle, 5000, *_graph(5000, 40_000, True), walks, 6, settings)


@pytest.mark.parametrize("walks", [114_688, 114_689, (1 << 18) + 1, 1 << 19, (1 << 19) + 1, 1 << 20, (1 << 20) + 1])
def test_many_walks_of_few_attempts(oracle, walks):
    _check(oracle, 5000, *_graph(5000, 40_000, True), walks, 5, ((1.0, 0.5), FEW))


@pytest.mark.parametrize("walks", [229_376, 229_377, (1 << 19) + 1, (1 << 20) + 1])
def test_few_attempts_on_more_entries(oracle, walks):
    _check(oracle, 5000, *_graph(5000, (1 << 21) + 5, True), walks, 3, ((1.0, 0.5), FEW))


@pytest.mark.parametrize("n,edges", [(1, [(0, 0)]), (2, [(0, 1), (1, 0)]), (2, [(0, 0), (0, 1), (1, 0)]),
                                     (3, [(0, 1), (1, 0), (1, 2)]), (2, [(0, 0), (0, 1), (1, 0), (1, 1)])])
@pytest.mark.parametrize("walks", [3, 200_000])
def test_tiny_graphs(oracle, n, edges, walks):
    src, dst = (np.array(c, dtype=np.int32) for c in zip(*edges))
    _check(oracle, n, src, dst, walks, 20 if walks < 100 else 4, (MANY, FEW, (1.0, 1.0)))


@pytest.mark.parametrize("weighted", [False, True])
def test_positions_beyond_31_bits(oracle, weighted):
    """Node 0, to which no edge leads, has 2^31 entries; the rows of the other nodes lie behind them."""
    from paper_2407_15452_amd import binding as gs
    n, first = 700, 1 << 31
    rng = np.random.default_rng(5)
    src, dst = (rng.integers(1, n, 9000).astype(np.int32) for _ in range(2))
    w = rng.lognormal(0, 1, src.size).astype(np.float32)
    off, nb, ww = oracle.csr_build(src, dst, w, n, 0)
    table = oracle.alias_build(off, ww)
    shifted = off.astype(np.int64) + first
    shifted[0] = 0

    def behind(a):
        out = torch.zeros(first + a.size, dtype=torch.as_tensor(a).dtype, device=DEV)
        out[first:] = _dev(a)
        return out

    g = gs.Csr(_dev(shifted), behind(nb))
    a = gs.Alias(behind(table[0]), behind(table[1])) if weighted else None
    for walks, p, q in ((1000, 0.5, 2.0), (20_000, 1.0, 0.5), (170_000, 0.5, 2.0), (170_000, 2.0, 1.0)):
        starts = (np.arange(walks) % (n - 1) + 1).astype(np.int32)
        want = oracle.node2vec_walk(off, nb, starts, 6, p, q, 11, alias=table if weighted else None)
        got = gs.gs_node2vec_walk(g, a, _dev(starts), 6, p, q, 11)
        np.testing.assert_array_equal(got.cpu().numpy(), want)
