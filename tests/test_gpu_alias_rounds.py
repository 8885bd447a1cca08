"""Alias tables whose smalls outnumber their larges for many rounds (skewed weights): the rounds that a workgroup, or
one wave of it, runs from registers, alone in a call (after the chip's rounds) and as rows of a graph; sums that any order
gives and sums that only the index order gives; bit for bit against the sequential construction."""
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


def _weights(kind, n, rng):
    if kind == "degrees":             # degree**0.75 of a skewed graph; isolated nodes weigh nothing
        return (np.floor(rng.pareto(1.1, n) * 2) ** 0.75).astype(np.float32)
    if kind == "steep":               # a handful of hubs takes nearly everything
        return (rng.pareto(0.5, n) + 0.1).clip(max=1e12).astype(np.float32)
    if kind == "hubs":                # `few` equal larges for most of the rounds, dropping out all at once
        w = np.full(n, 0.5, dtype=np.float32)
        w[rng.choice(n, max(1, n // 100), replace=False)] = 40.0
        return w
    return rng.lognormal(0, 1, n).astype(np.float32)


@pytest.mark.parametrize("kind", ["degrees", "steep", "hubs", "lognormal"])
@pytest.mark.parametrize("n", [(1 << 17) + 5, 400_003, (3 << 19) + 1])       # 16 and 32 rounds of the chip
def test_alone(oracle, kind, n):
    w = _weights(kind, n, np.random.default_rng(n))
    _check(oracle, np.array([0, n], dtype=np.int64), w)


@pytest.mark.parametrize("n", [(1 << 22) + 5, 1 << 26, (1 << 26) + 1])       # 256 threads a workgroup up to 2^26 entries
def test_alone_and_very_long(oracle, n):
    _check(oracle, np.array([0, n], dtype=np.int64), _weights("lognormal", n, np.random.default_rng(n)))


@pytest.mark.parametrize("larges", [1, 63, 64, 65, 2047, 2048, 2049, 8191, 8192])
def test_alone_with_so_many_larges(oracle, larges):
    """Equal larges that last for 20 rounds and more of 300,000 smalls."""
    n = 300_000
    w = np.full(n, 1.0, dtype=np.float32)
    rng = np.random.default_rng(larges)
    w += (rng.random(n) * 0.1).astype(np.float32)
    w[rng.choice(n, larges, replace=False)] = 1.0e6 / larges
    _check(oracle, np.array([0, n], dtype=np.int32), w)


@pytest.mark.parametrize("kind", ["degrees", "steep", "hubs", "lognormal"])
@pytest.mark.parametrize("dtype", [np.int32, np.int64])
def test_rows(oracle, kind, dtype):
    rng = np.random.default_rng(7)
    lens = np.concatenate([[50_000, 20_000, 9000, 3071, 3072, 3073, 2049, 2050, 1024, 1025, 256, 257],
                           rng.integers(0, 40, 3000), rng.integers(200, 2600, 60)])
    seg = np.concatenate([[0], np.cumsum(lens)]).astype(dtype)
    _check(oracle, seg, _weights(kind, int(seg[-1]), rng))


def test_order_of_the_sum_matters(oracle):
    """Weights over too many binades for an exact sum, in segments of every size class."""
    rng = np.random.default_rng(11)
    for n in (20, 100, 700, 2000, 5000, 140_000):
        w = np.exp(12 * rng.standard_normal(n)).astype(np.float32)
        _check(oracle, np.array([0, n], dtype=np.int64), w)
        _check(oracle, np.array([0, 0, n - 3, n], dtype=np.int64), w)
    w = np.zeros(3000, dtype=np.float32)                      # all zero; denormals
    _check(oracle, np.array([0, 3000], dtype=np.int64), w)
    w[::7] = np.float32(1e-42)
    w[5] = 1.0
    _check(oracle, np.array([0, 3000], dtype=np.int64), w)


@pytest.mark.parametrize("segments", [1, 15, 16, 17, 1025, 16_385, 600_001])
def test_rows_of_all_sizes_side_by_side(oracle, segments):
    """The launch that takes rows by waves and by workgroups: 16 to 512 segments per workgroup, sizes at its edges, many long
    rows next to each other, and none."""
    rng = np.random.default_rng(segments)
    edges = [32, 33, 255, 256, 257, 1023, 1024, 1025, 2047, 2048, 2049, 0, 1]
    lens = rng.integers(0, 12, segments)
    some = rng.random(segments) < min(1.0, 2000 / segments)
    lens[some] = rng.choice(edges, int(some.sum()))
    for long_rows in (True, False):
        use = lens if long_rows else np.minimum(lens, 300 if segments > 1 else 1024)
        seg = np.concatenate([[0], np.cumsum(use)]).astype(np.int32)
        if seg[-1] > 0:
            _check(oracle, seg, _weights("steep" if long_rows else "lognormal", int(seg[-1]), rng))
