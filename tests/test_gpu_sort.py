"""The device radix sort through the calls that use it: tile edges (2048 and 8192 records), the
size from which the large tiles are taken (2^21), and odd and even numbers of passes."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module")
def gs():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2407_15452_amd import binding
    binding.lib()
    return binding


def _t(a):
    return torch.as_tensor(np.ascontiguousarray(a)).to(DEV)


@pytest.mark.parametrize("n", [1, 2047, 2048, 2049, (1 << 21) - 1, (1 << 21) + 8191])
@pytest.mark.parametrize("num_nodes", [1, 200, 60_000, 5_000_000, (1 << 31) - 1])    # 1, 1, 2, 3 and 4 passes
def test_sort_pairs_sizes(gs, n, num_nodes):
    rng = np.random.default_rng(n + num_nodes)
    c = rng.integers(0, num_nodes, n).astype(np.int32)
    c[rng.integers(0, n, n // 3)] = c[0]                   # one long run of equal sources
    c[rng.integers(0, n, n // 50)] = -7                    # not rows: last, in input order
    o = np.arange(n, dtype=np.int32)                       # shows whether the order is stable
    at = np.argsort(np.where(c < 0, num_nodes, c.astype(np.int64)), kind="stable")
    got_c, got_o = gs.gs_sort_pairs(_t(c), _t(o), num_nodes)
    np.testing.assert_array_equal(got_o.cpu().numpy(), o[at])
    np.testing.assert_array_equal(got_c.cpu().numpy(), c[at])


@pytest.mark.parametrize("n", [8191, 8192, (3 << 19) - 1, (3 << 19) + 4095, (5 << 20) - 1, (5 << 20) + 1])
@pytest.mark.parametrize("num_nodes", [(1 << 18) - 1, (1 << 20) - 1])                # two passes of 9 and of 10 bits
def test_sort_pairs_in_wide_digits(gs, n, num_nodes):
    """Both sides of every size of tile, and digits of 8 bits where the workspace leaves room for no more."""
    rng = np.random.default_rng(n + num_nodes)
    c = rng.integers(0, num_nodes, n).astype(np.int32)
    c[rng.integers(0, n, n // 3)] = c[0]
    c[rng.integers(0, n, n // 50)] = num_nodes + 3
    o = np.arange(n, dtype=np.int32)
    at = np.argsort(np.minimum(c, num_nodes), kind="stable")
    size = gs.gs_sort_pairs_workspace_bytes(n)
    tiles = max(min(n, (1 << 21) - 1) // 2048, n // 8192) + 1
    narrow = 2 * (-(-4 * n // 256) * 256) + 1024 * tiles + 1024
    for room in {size, min(size, narrow)}:
        got_c, got_o = gs.gs_sort_pairs(_t(c), _t(o), num_nodes, ws=torch.empty(room, dtype=torch.uint8, device=DEV))
        np.testing.assert_array_equal(got_o.cpu().numpy(), o[at])
        np.testing.assert_array_equal(got_c.cpu().numpy(), c[at])


@pytest.mark.parametrize("n,num_nodes", [(1 << 20, 60_000), ((1 << 20) + 1, 60_000), ((3 << 19) - 1, 60_000), (3 << 20, 60_000), ((3 << 20) + 1, 60_000), (1 << 19, (1 << 20) - 1), ((1 << 19) + 1, (1 << 20) - 1),
                                         (300_001, 60_000), (300_001, 3), (40_000, 2)])
def test_sort_pairs_of_few_tiles(gs, n, num_nodes):
    """Both sides of the most counts that the scan for few tiles takes: 768 tiles of 256 digits, 256 of 1024; digits of one and two bits."""
    test_sort_pairs_sizes(gs, n, num_nodes)


@pytest.mark.parametrize("m,num_nodes", [(1, 1), (1023, 9), (1024, 300), (40_000, 5000), (40_001, 70_000),
                                         ((1 << 20) + 17, 3_000_000)])     # 1, 2, 3, 4, 5 and 6 passes
@pytest.mark.parametrize("weighted", [False, True])
def test_csr_sizes(gs, oracle, m, num_nodes, weighted):
    rng = np.random.default_rng(m)
    src = rng.integers(-1, num_nodes + 1, m).astype(np.int32)
    dst = rng.integers(0, num_nodes, m).astype(np.int32)
    dup = rng.integers(0, m, m // 4)
    src[dup], dst[dup] = src[0], dst[0]                    # one entry many times over
    w = rng.random(m).astype(np.float32) if weighted else None
    flags = gs.GS_SYMMETRIZE | gs.GS_DEDUPE
    off, nb, wo = oracle.csr_build(src, dst, w, num_nodes, flags, 32)
    g = gs.gs_csr_build(_t(src), _t(dst), _t(w) if weighted else None, num_nodes, flags)
    np.testing.assert_array_equal(g.offsets.cpu().numpy(), off)
    np.testing.assert_array_equal(g.nbrs.cpu().numpy(), nb)
    if weighted:
        np.testing.assert_array_equal(g.weights.cpu().numpy(), wo)


@pytest.mark.parametrize("n,num_nodes", [(1, 1 << 20), (2049, 1 << 24), (5000, (1 << 31) - 1)])
def test_unique_ids_by_sorting(gs, n, num_nodes):
    """Graphs far larger than the batch: the ids are sorted (3 and 4 passes)."""
    rng = np.random.default_rng(n)
    ids = rng.integers(0, num_nodes, n).astype(np.int32)
    ids[rng.integers(0, n, n // 2)] = ids[0]
    ids[rng.integers(0, n, n // 10)] = -1
    want, inverse = np.unique(ids[ids >= 0], return_inverse=True)
    u, count, inv = gs.gs_unique_ids(_t(ids), num_nodes)
    assert int(count.item()) == want.size
    np.testing.assert_array_equal(u.cpu().numpy()[:want.size], want)
    got = inv.cpu().numpy()
    np.testing.assert_array_equal(got[ids >= 0], inverse)
    assert (got[ids < 0] == -1).all()


@pytest.mark.parametrize("num_nodes", [1, 2, 3, 255, 256, 257, 65_535, 65_536])
@pytest.mark.parametrize("weighted", [False, True])
def test_csr_with_nodes_that_fill_their_bits(gs, oracle, num_nodes, weighted):
    """Dropped records (ids that are no nodes, self loops) next to the largest entry a graph can have."""
    m = 5000
    rng = np.random.default_rng(num_nodes)
    src, dst = (rng.integers(-1, num_nodes + 1, m).astype(np.int32) for _ in range(2))
    src[:3], dst[:3] = num_nodes - 1, [num_nodes - 1, max(0, num_nodes - 2), num_nodes - 1]
    w = rng.random(m).astype(np.float32) if weighted else None
    for flags in (0, gs.GS_SYMMETRIZE | gs.GS_DROP_SELF_LOOPS | gs.GS_DEDUPE):
        off, nb, wo = oracle.csr_build(src, dst, w, num_nodes, flags, 32)
        g = gs.gs_csr_build(_t(src), _t(dst), _t(w) if weighted else None, num_nodes, flags)
        np.testing.assert_array_equal(g.offsets.cpu().numpy(), off)
        np.testing.assert_array_equal(g.nbrs.cpu().numpy(), nb)
        if weighted:
            np.testing.assert_array_equal(g.weights.cpu().numpy(), wo)


@pytest.mark.parametrize("walks", [1, 1023, 1024, 1025, 70_001, (4096 << 10) - 1, (4096 << 10) + 1])
def test_offsets_of_pairs(gs, walks):
    """The 64-bit scan: one tile, tiles whose sums every workgroup adds up, and more tiles than that."""
    length = np.random.default_rng(walks).integers(1, 4, walks)
    w = np.where(np.arange(3)[None, :] < length[:, None], 7, -1).astype(np.int32)
    want = np.concatenate([[0], np.cumsum(2 * (length - 1))])            # window 1: both directions of every step
    np.testing.assert_array_equal(gs.gs_pair_offsets(_t(w), 1).cpu().numpy(), want)
