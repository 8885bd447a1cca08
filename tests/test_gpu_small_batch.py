"""The two-launch step of small batches against the CPU reference: the largest batch that takes it
and the first that does not, rows just below and above the length at which a whole workgroup sums
them, one row named by every term, and ids that overfill one workgroup's table or its terms."""
import numpy as np
import pytest
import torch

from tolerances import LOSS_RTOL, assert_emb_close, assert_half_close

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _step(oracle, n, dim, c, o, neg, lr=0.05):
    from paper_2407_15452_amd import binding as gs, inputs
    w_in, w_out = inputs.random_tables(n, dim, 5, 0.4)
    d_in, d_out = w_in.to(DEV), w_out.to(DEV)
    t = [torch.as_tensor(np.ascontiguousarray(x)).to(DEV) for x in (c, o, neg)]
    loss = gs.gs_sgns_step(d_in, d_out, *t, lr)
    h_in, h_out = w_in.numpy().copy(), w_out.numpy().copy()
    want = oracle.sgns_step(h_in, h_out, c, o, neg, lr)
    assert abs(float(loss.item()) - want) <= LOSS_RTOL * abs(want)
    assert_emb_close(d_in.cpu().numpy(), h_in)
    assert_emb_close(d_out.cpu().numpy(), h_out)


@pytest.mark.parametrize("b,k,dim", [(1, 0, 4), (2, 1, 256), (7021, 5, 12), (7022, 5, 12), (24576, 0, 8),
                                     (24577, 0, 8), (792, 60, 16), (1000, 3, 260)])
def test_sizes(oracle, b, k, dim):
    _sizes(oracle, 20_000, b, k, dim)


@pytest.mark.parametrize("n", [127, 128])
def test_few_nodes(oracle, n):
    """4096 ids: the square is 2^17 times 128."""
    _sizes(oracle, n, 1024, 2, 16)


def _sizes(oracle, n, b, k, dim):
    rng = np.random.default_rng(b + k)
    c = np.repeat(rng.integers(0, n, (b + 6) // 7), 7)[:b].astype(np.int32)
    o = rng.integers(0, n, b).astype(np.int32)
    neg = rng.integers(0, n, (b, k)).astype(np.int32)
    _step(oracle, n, dim, c, o, neg)


@pytest.mark.parametrize("run", [63, 64, 65, 129, 4000])
def test_long_rows(oracle, run):
    """`run` terms name one context row, and `run` separate runs one input row."""
    rng = np.random.default_rng(run)
    n, b, k = 5000, 4000, 2
    c = np.arange(b, dtype=np.int32) % n
    c[:2 * run:2] = 17
    o = rng.integers(100, n, b).astype(np.int32)
    o[rng.permutation(b)[:run]] = 4
    neg = rng.integers(100, n, (b, k)).astype(np.int32)
    _step(oracle, n, 20, c, o, neg, 0.01)


@pytest.mark.parametrize("distinct,b", [(1500, 2000), (900, 4000)])
def test_ids_that_share_a_hash(oracle, distinct, b):
    """Ids that one workgroup owns: more than its table holds, and more terms than it keeps."""
    n = 500_000
    ids = np.arange(n, dtype=np.uint64)
    owned = np.nonzero(((ids * 2654435761) & 0xFFFFFFFF) >> 24 == 3)[0]
    assert owned.size >= distinct
    rng = np.random.default_rng(b)
    pick = owned[:distinct]
    o = pick[rng.integers(0, distinct, b)].astype(np.int32)
    neg = pick[rng.integers(0, distinct, (b, 1))].astype(np.int32)
    c = rng.integers(0, n, b).astype(np.int32)
    _step(oracle, n, 4, c, o, neg)


@pytest.mark.parametrize("dim,b,k", [(8, 3000, 3), (200, 1500, 5), (512, 700, 2)])
@pytest.mark.parametrize("fmt", ["bf16", "f16"])
def test_sixteen_bit_tables(oracle, dim, b, k, fmt):
    """Short rows and two long ones, in rows of up to 256, 512 and 1024 bytes."""
    from paper_2407_15452_amd import binding as gs, inputs
    n = 20_000
    rng = np.random.default_rng(dim)
    tabs = [t.to(torch.bfloat16 if fmt == "bf16" else torch.float16) for t in inputs.random_tables(n, dim, 5, 0.4)]
    dev = [t.to(DEV) for t in tabs]
    host = [t.view(torch.int16).numpy().view(np.uint16).copy() for t in tabs]
    c = np.repeat(rng.integers(0, n, b // 4 + 1), 4)[:b].astype(np.int32)
    c[:300:2] = 17
    o = rng.integers(0, n, b).astype(np.int32)
    o[:129] = 4
    neg = rng.integers(0, n, (b, k)).astype(np.int32)
    want = oracle.sgns_step(*host, c, o, neg, 0.02, dtype=oracle.BF16 if fmt == "bf16" else oracle.F16)
    loss = gs.gs_sgns_step(*dev, *(torch.as_tensor(x).to(DEV) for x in (c, o, neg)), 0.02)
    assert abs(float(loss.item()) - want) <= LOSS_RTOL * abs(want)
    for d, h in zip(dev, host):
        assert_half_close(d.view(torch.int16).cpu().numpy().view(np.uint16), h, fmt)
