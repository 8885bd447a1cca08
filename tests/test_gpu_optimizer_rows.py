"""Momentum and Adam iterations where rows inside and outside the batch take different kernels:
counters per vertex, a table of the batch's input keys, a table of all its keys (how a row outside
the batch is told), with rows of one term, long rows and rows no batch names."""
import numpy as np
import pytest
import torch

from tolerances import EMB_ATOL, LOSS_RTOL, assert_emb_close, assert_half_close

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
# (nodes, pairs, negatives, columns): per-vertex counters; input keys in a table; all keys in a table; tables that no cache
# holds (more than 256 MB in bf16 too), rows that fill a workgroup's lanes and rows that do not
SHAPES = [(3_000, 9_000, 5, 20), (400_000, 9_000, 5, 8), (800_000, 9_000, 5, 8), (280_000, 9_000, 3, 128), (430_000, 9_000, 3, 104)]


def _batch(n, b, k, seed):
    rng = np.random.default_rng(seed)
    c = np.repeat(rng.integers(0, n, b // 4 + 1), 4)[:b].astype(np.int32)
    c[::3] = 11
    o = rng.integers(0, n, b).astype(np.int32)
    o[::4] = n - 1                                          # a long row in each table
    return c, o, rng.integers(0, n, (b, k)).astype(np.int32)


def _dev(a):
    return torch.as_tensor(np.ascontiguousarray(a)).to(DEV)


@pytest.mark.parametrize("n,b,k,dim", SHAPES)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_momentum(oracle, n, b, k, dim, dtype):
    from paper_2407_15452_amd import binding as gs, inputs
    dim = dim if dtype == "f32" else 8 * ((dim + 7) // 8)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    tabs = [t.to(tdt) for t in (*inputs.random_tables(n, dim, 3, 0.3), *inputs.random_tables(n, dim, 4, 0.05))]
    host = [t.numpy().copy() if dtype == "f32" else t.view(torch.int16).numpy().view(np.uint16).copy() for t in tabs]
    dev = [t.to(DEV) for t in tabs]
    c, o, neg = _batch(n, b, k, n)
    lr, mu = 0.01, 0.875
    want = oracle.sgns_momentum_step(*host, c, o, neg, lr, mu, dtype=oracle.F32 if dtype == "f32" else oracle.BF16)
    loss = gs.gs_sgns_momentum_step(*dev, _dev(c), _dev(o), _dev(neg), lr, mu)
    assert abs(float(loss.item()) - want) <= LOSS_RTOL * abs(want)
    for d, h in zip(dev, host):
        if dtype == "f32":
            assert_emb_close(d.cpu().numpy(), h)
        else:
            assert_half_close(d.view(torch.int16).cpu().numpy().view(np.uint16), h, dtype)


@pytest.mark.parametrize("n,b,k,dim", SHAPES)
def test_adam(oracle, n, b, k, dim):
    from paper_2407_15452_amd import binding as gs, inputs
    w, m = inputs.random_tables(n, dim, 3, 0.3), inputs.random_tables(n, dim, 4, 0.05)
    v = [t.abs() + 0.01 for t in inputs.random_tables(n, dim, 5, 0.1)]   # (denominators well above zero)
    host = [t.numpy().copy() for t in (*w, *m, *v)]
    dev = [torch.as_tensor(h).to(DEV) for h in host]
    c, o, neg = _batch(n, b, k, n)
    want = oracle.sgns_adam_step(*host, c, o, neg, 0.01, 0.9, 0.999, 1e-8, 5)
    loss = gs.gs_sgns_adam_step(*dev, _dev(c), _dev(o), _dev(neg), 0.01, 0.9, 0.999, 1e-8, 5)
    assert abs(float(loss.item()) - want) <= LOSS_RTOL * abs(want)
    for i, (d, h) in enumerate(zip(dev, host)):
        got = d.cpu().numpy()
        if i < 2:
            assert np.abs(got - h).max() <= EMB_ATOL
        else:
            assert (np.abs(got - h) <= 1e-6 + 1e-5 * np.abs(h)).all()


def test_adam_without_pairs(oracle):
    from paper_2407_15452_amd import binding as gs, inputs
    n, dim = 777, 12
    host = [t.numpy().copy() for s in (1, 2, 3) for t in inputs.random_tables(n, dim, s, 0.2)]
    for h in host[4:]:
        np.abs(h, out=h)
        h += 0.01
    dev = [torch.as_tensor(h).to(DEV) for h in host]
    none = np.zeros(0, dtype=np.int32)
    oracle.sgns_adam_step(*host, none, none, none.reshape(0, 2), 0.01, 0.9, 0.999, 1e-8, 5)
    gs.gs_sgns_adam_step(*dev, _dev(none), _dev(none), _dev(none.reshape(0, 2)), 0.01, 0.9, 0.999, 1e-8, 5)
    for d, h in zip(dev, host):
        assert np.abs(d.cpu().numpy() - h).max() <= 1e-6
