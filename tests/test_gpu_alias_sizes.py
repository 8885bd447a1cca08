"""Alias tables at the sizes where another kernel takes over (one lane up to 32 entries, one wave up
to 256 and up to 2048, a workgroup beyond, the whole chip for a single segment of 2^17), and the index-order sum and the narrow stretches of long
segments on weights that make them hard; bit for bit against the sequential construction."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _check(oracle, seg, w):
    from paper_2407_15452_amd import binding as gs
    prob, alias = oracle.alias_build(seg, w)
    a = gs.gs_alias_build(torch.as_tensor(seg).to(DEV), torch.as_tensor(w).to(DEV))
    np.testing.assert_array_equal(a.alias.cpu().numpy(), alias)
    np.testing.assert_array_equal(a.prob.cpu().numpy(), prob)


@pytest.mark.parametrize("dtype", [np.int32, np.int64])
def test_segment_sizes(oracle, dtype):
    rng = np.random.default_rng(9)
    lens = np.concatenate([[1, 2, 31, 32, 33, 63, 64, 65, 255, 256, 257, 1023, 2047, 2048, 2049, 4096, 4097, 0],
                           rng.integers(0, 300, 40_000)])
    seg = np.concatenate([[0], np.cumsum(lens)]).astype(dtype)
    w = rng.lognormal(0, 2.0, int(seg[-1])).astype(np.float32)
    w[rng.random(w.size) < 0.1] = 0
    _check(oracle, seg, w)


@pytest.mark.parametrize("n", [2, 32, 33, 256, 257, 2048])
def test_one_short_segment(oracle, n):
    w = np.random.default_rng(n).random(n).astype(np.float32)
    _check(oracle, np.array([0, n], dtype=np.int32), w)


@pytest.mark.parametrize("kind", ["ties", "wide", "tenths", "few_small", "two_hubs", "alternating"])
@pytest.mark.parametrize("n", [2049, 4096, (1 << 17) - 1, 1 << 17, 500_001])
def test_long_segments(oracle, kind, n):
    rng = np.random.default_rng(n)
    if kind == "ties":              # the running sum's unit is twice the last bit of every further weight
        w = (rng.integers(0, 1 << 23, n).astype(np.uint32) | 0x3f800001).view(np.float32).copy()
        w[0] = 2.0 ** 30
    elif kind == "wide":            # weights over 200 binades
        w = np.exp(15 * rng.standard_normal(n)).astype(np.float32)
    elif kind == "tenths":          # equal weights whose sum rounds
        w = np.full(n, 0.1, dtype=np.float32)
    elif kind == "few_small":       # short list of smalls, long list of larges
        w = np.full(n, 1.0, dtype=np.float32)
        w[::997] = 0.99
    elif kind == "two_hubs":        # two entries absorb all others
        w = np.full(n, 1e-3, dtype=np.float32)
        w[7], w[n - 2] = 4e4, 3e4
    else:                           # most iterations turn their large into a small
        w = np.where(np.arange(n) % 3 == 0, 1.5, 0.75).astype(np.float32)
    _check(oracle, np.array([0, n], dtype=np.int64), w)


def test_long_segment_in_a_smaller_workspace(oracle):
    """A workspace of the size that several segments need: the single segment is built by one workgroup."""
    from paper_2407_15452_amd import binding as gs
    import ctypes as C
    n = 200_003
    w = np.random.default_rng(4).lognormal(0, 1.5, n).astype(np.float32)
    seg = np.array([0, n], dtype=np.int64)
    prob, alias = oracle.alias_build(seg, w)
    size = gs.lib().gs_alias_build_workspace_bytes(C.c_int64(2), C.c_int64(n))
    assert size < gs.lib().gs_alias_build_workspace_bytes(C.c_int64(1), C.c_int64(n))
    a = gs.gs_alias_build(torch.as_tensor(seg).to(DEV), torch.as_tensor(w).to(DEV),
                          ws=torch.empty(size, dtype=torch.uint8, device=DEV))
    np.testing.assert_array_equal(a.alias.cpu().numpy(), alias)
    np.testing.assert_array_equal(a.prob.cpu().numpy(), prob)
