"""GPU parity: every C-ABI entry point of libgs.so against the CPU oracle.

Integer outputs (CSR, alias indices, walks, pairs, negatives) must be
bit-identical; alias probabilities are bit-identical too because the
construction order is part of the definition.  The SGNS step must agree within
1e-5 (relative for the loss, max-abs for the embeddings).
"""
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
    binding.lib()          # raises if libgs.so was not built
    return binding


@pytest.fixture(scope="module")
def cfg0(gs, oracle):
    """Workload 0: edge list, oracle CSR, device CSR."""
    from paper_2407_15452_amd import inputs
    wl = inputs.WORKLOADS[0]
    src, dst, _ = inputs.edge_list(wl, "cpu")
    flags = oracle.SYMMETRIZE | oracle.DROP_SELF_LOOPS | oracle.DEDUPE
    off, nb, _ = oracle.csr_build(src.numpy(), dst.numpy(), None, wl.num_nodes, flags)
    g = gs.gs_csr_build(src.to(DEV), dst.to(DEV), None, wl.num_nodes, flags)
    torch.cuda.synchronize()
    return wl, (off, nb), g


def _t(a, dtype=None):
    t = torch.as_tensor(np.ascontiguousarray(a))
    if dtype is not None:
        t = t.to(dtype)
    return t.to(DEV)


# ----------------------------------------------------------------------------- CSR
@pytest.mark.parametrize("flags", range(8))
@pytest.mark.parametrize("bits", [32, 64])
def test_csr_build(gs, oracle, flags, bits):
    rng = np.random.default_rng(1000 + flags)
    n, m = 5000, 61_237                        # 30+ sort tiles and a ragged tail
    src = rng.integers(-2, n + 2, m).astype(np.int32)
    dst = rng.integers(-2, n + 2, m).astype(np.int32)
    dup = rng.integers(0, m, m // 4)            # plenty of duplicates
    src[dup], dst[dup] = src[(dup * 7) % m], dst[(dup * 7) % m]
    w = rng.random(m).astype(np.float32)
    off, nb, wo = oracle.csr_build(src, dst, w, n, flags, bits)
    g = gs.gs_csr_build(_t(src), _t(dst), _t(w), n, flags, bits)
    assert g.num_entries == nb.size
    np.testing.assert_array_equal(g.offsets.cpu().numpy(), off)
    np.testing.assert_array_equal(g.nbrs.cpu().numpy(), nb)
    np.testing.assert_array_equal(g.weights.cpu().numpy(), wo)


def test_csr_build_workload0_and_empty(gs, oracle, cfg0):
    wl, (off, nb), g = cfg0
    assert nb.size == 2 * wl.num_edges
    np.testing.assert_array_equal(g.offsets.cpu().numpy(), off)
    np.testing.assert_array_equal(g.nbrs.cpu().numpy(), nb)
    e = torch.zeros(0, dtype=torch.int32, device=DEV)
    g0 = gs.gs_csr_build(e, e, None, 7, 7)
    assert g0.num_entries == 0 and (g0.offsets == 0).all()


def test_csr_build_rejects_bad_arguments(gs):
    e = torch.zeros(4, dtype=torch.int32, device=DEV)
    with pytest.raises(gs.GsError):
        gs.gs_csr_build(e, e, None, 4, 0, offset_bits=16)
    with pytest.raises(gs.GsError):
        gs.gs_csr_build(e, e, None, 4, 64)
    with pytest.raises(gs.GsError) as ei:
        gs.gs_csr_build(e, e, None, 4, 0, ws=torch.empty(256, dtype=torch.uint8, device=DEV))
    assert ei.value.status == gs.GS_EWORKSPACE


# ----------------------------------------------------------------------------- alias
def test_alias_build_per_row_and_single_segment(gs, oracle, cfg0):
    wl, (off, nb), g = cfg0
    rng = np.random.default_rng(7)
    w = rng.lognormal(0, 1, nb.size).astype(np.float32)
    w[rng.random(nb.size) < 0.05] = 0
    prob, alias = oracle.alias_build(off, w)
    a = gs.gs_alias_build(g.offsets, _t(w))
    np.testing.assert_array_equal(a.alias.cpu().numpy(), alias)
    np.testing.assert_array_equal(a.prob.cpu().numpy(), prob)
    # one long segment (the noise table), 64-bit segment offsets
    deg = np.diff(off).astype(np.float64)
    nw = np.where(deg > 0, deg ** 0.75, 0).astype(np.float32)
    seg = np.array([0, nw.size], dtype=np.int64)
    prob, alias = oracle.alias_build(seg, nw)
    a = gs.gs_alias_build(_t(seg), _t(nw))
    np.testing.assert_array_equal(a.alias.cpu().numpy(), alias)
    np.testing.assert_array_equal(a.prob.cpu().numpy(), prob)


# ----------------------------------------------------------------------------- walks
def _walk_inputs(wl, count, first=0):
    from paper_2407_15452_amd import inputs
    return inputs.walk_starts(wl.num_nodes, first, count, "cpu")


def test_random_walk_workload0(gs, oracle, cfg0):
    wl, (off, nb), g = cfg0
    nw = wl.num_nodes * wl.walks_per_node
    starts = _walk_inputs(wl, nw)
    want = oracle.random_walk(off, nb, starts.numpy(), wl.walk_len, wl.walk_seed)
    got = gs.gs_random_walk(g, None, starts.to(DEV), wl.walk_len, wl.walk_seed)
    np.testing.assert_array_equal(got.cpu().numpy(), want)
    assert (want == -1).any()                   # isolated starts exist: dead walks covered
    # a sub-range on its own, odd length, odd count
    part = gs.gs_random_walk(g, None, starts[1001:1001 + 777].to(DEV), wl.walk_len, wl.walk_seed,
                             walk_id_base=1001)
    np.testing.assert_array_equal(part.cpu().numpy(), want[1001:1001 + 777])


@pytest.mark.parametrize("walk_len", [1, 2, 16, 17, 33])
def test_random_walk_lengths_weighted_int64(gs, oracle, cfg0, walk_len):
    wl, (off, nb), g = cfg0
    rng = np.random.default_rng(walk_len)
    w = (rng.random(nb.size) + 0.05).astype(np.float32)
    table = oracle.alias_build(off, w)
    a = gs.gs_alias_build(g.offsets, _t(w))
    starts = rng.integers(-1, wl.num_nodes + 1, 3001).astype(np.int32)   # includes invalid starts
    want = oracle.random_walk(off, nb, starts, walk_len, 99, alias=table, walk_id_base=1 << 40)
    got = gs.gs_random_walk(g, a, _t(starts), walk_len, 99, walk_id_base=1 << 40)
    np.testing.assert_array_equal(got.cpu().numpy(), want)
    g64 = gs.Csr(g.offsets.to(torch.int64), g.nbrs)
    got = gs.gs_random_walk(g64, a, _t(starts), walk_len, 99, walk_id_base=1 << 40)
    np.testing.assert_array_equal(got.cpu().numpy(), want)


def test_walks_on_directed_graph_with_sinks(gs, oracle):
    rng = np.random.default_rng(5)
    n, m = 3000, 6000
    src = rng.integers(0, n, m).astype(np.int32)
    dst = rng.integers(0, n, m).astype(np.int32)
    flags = oracle.DROP_SELF_LOOPS | oracle.DEDUPE
    off, nb, _ = oracle.csr_build(src, dst, None, n, flags)
    g = gs.gs_csr_build(_t(src), _t(dst), None, n, flags)
    starts = (np.arange(9000) % n).astype(np.int32)
    want = oracle.random_walk(off, nb, starts, 12, 3)
    got = gs.gs_random_walk(g, None, _t(starts), 12, 3)
    np.testing.assert_array_equal(got.cpu().numpy(), want)
    want = oracle.node2vec_walk(off, nb, starts, 12, 0.5, 2.0, 3)
    got = gs.gs_node2vec_walk(g, None, _t(starts), 12, 0.5, 2.0, 3)
    np.testing.assert_array_equal(got.cpu().numpy(), want)
    assert (want == -1).any()


@pytest.mark.parametrize("p,q", [(0.5, 2.0), (4.0, 0.25), (1.0, 1.0)])
def test_node2vec_walk_workload0(gs, oracle, cfg0, p, q):
    wl, (off, nb), g = cfg0
    nw = 20_011
    starts = _walk_inputs(wl, nw, first=123)
    want = oracle.node2vec_walk(off, nb, starts.numpy(), 30, p, q, wl.walk_seed, walk_id_base=123)
    got = gs.gs_node2vec_walk(g, None, starts.to(DEV), 30, p, q, wl.walk_seed, walk_id_base=123)
    np.testing.assert_array_equal(got.cpu().numpy(), want)
    if p == 1.0 and q == 1.0:
        first_order = gs.gs_random_walk(g, None, starts.to(DEV), 30, wl.walk_seed, walk_id_base=123)
        assert torch.equal(first_order, got)


def test_node2vec_walk_weighted(gs, oracle, cfg0):
    wl, (off, nb), g = cfg0
    rng = np.random.default_rng(11)
    w = rng.lognormal(0, 1, nb.size).astype(np.float32)
    table = oracle.alias_build(off, w)
    a = gs.gs_alias_build(g.offsets, _t(w))
    starts = _walk_inputs(wl, 10_000)
    want = oracle.node2vec_walk(off, nb, starts.numpy(), 25, 0.5, 2.0, 17, alias=table)
    got = gs.gs_node2vec_walk(g, a, starts.to(DEV), 25, 0.5, 2.0, 17)
    np.testing.assert_array_equal(got.cpu().numpy(), want)


def test_walk_argument_errors(gs, cfg0):
    wl, _, g = cfg0
    s = torch.zeros(4, dtype=torch.int32, device=DEV)
    with pytest.raises(gs.GsError):
        gs.gs_random_walk(g, None, s, 0, 1)
    with pytest.raises(gs.GsError):
        gs.gs_node2vec_walk(g, None, s, 5, 0.0, 1.0, 1)
    with pytest.raises(gs.GsError):
        gs.gs_node2vec_walk(g, None, s, 5, 1.0, float("nan"), 1)
    assert gs.gs_random_walk(g, None, s[:0], 5, 1).shape == (0, 5)


# ----------------------------------------------------------------------------- pairs / negatives
@pytest.mark.parametrize("walk_len,window", [(20, 5), (5, 3), (4, 7), (1, 2), (80, 10), (300, 2),
                                             (4096, 3), (2, 1), (64, 64)])
def test_make_pairs(gs, oracle, walk_len, window):
    rng = np.random.default_rng(walk_len * 31 + window)
    nw = 1500 if walk_len < 100 else 150
    walks = rng.integers(0, 10_000, (nw, walk_len)).astype(np.int32)
    for i in range(0, nw, 3):                  # a third of the walks end early
        walks[i, rng.integers(0, walk_len + 1):] = -1
    wc, wo = oracle.make_pairs(walks, window)
    c, o, n = gs.gs_make_pairs(_t(walks), window)
    assert n == wc.size
    np.testing.assert_array_equal(c.cpu().numpy(), wc)
    np.testing.assert_array_equal(o.cpu().numpy(), wo)


def test_make_pairs_empty_and_errors(gs):
    w = torch.zeros((0, 8), dtype=torch.int32, device=DEV)
    c, o, n = gs.gs_make_pairs(w, 3)
    assert n == 0
    dead = torch.full((5, 8), -1, dtype=torch.int32, device=DEV)
    assert gs.gs_make_pairs(dead, 3)[2] == 0
    with pytest.raises(gs.GsError):
        gs.gs_make_pairs(dead, 0)


def test_sample_negatives(gs, oracle, cfg0):
    wl, (off, nb), g = cfg0
    from paper_2407_15452_amd import inputs
    nw = inputs.noise_weights(torch.as_tensor(off)).numpy()
    seg = np.array([0, wl.num_nodes], dtype=np.int32)
    table = oracle.alias_build(seg, nw)
    a = gs.gs_alias_build(_t(seg), _t(nw))
    want = oracle.sample_negatives(table, wl.num_nodes, 70_001, wl.num_neg, wl.neg_seed,
                                   pair_index_base=(1 << 35) + 3)
    got = gs.gs_sample_negatives(a, wl.num_nodes, 70_001, wl.num_neg, wl.neg_seed,
                                 pair_index_base=(1 << 35) + 3)
    np.testing.assert_array_equal(got.cpu().numpy(), want)
    want = oracle.sample_negatives(None, 977, 5000, 3, 5)
    got = gs.gs_sample_negatives(None, 977, 5000, 3, 5, device=DEV)
    np.testing.assert_array_equal(got.cpu().numpy(), want)


# ----------------------------------------------------------------------------- SGNS
from tolerances import EMB_ATOL, LOSS_RTOL, assert_emb_close, assert_half_close  # noqa: E402


def _sgns_case(gs, oracle, w_in, w_out, c, o, neg, lr):
    d_in, d_out = w_in.to(DEV), w_out.to(DEV)
    loss = gs.gs_sgns_step(d_in, d_out, _t(c), _t(o), _t(neg), lr)
    torch.cuda.synchronize()
    h_in, h_out = w_in.numpy().copy(), w_out.numpy().copy()
    want = oracle.sgns_step(h_in, h_out, c, o, neg, lr)
    got = float(loss.item())
    assert abs(got - want) <= LOSS_RTOL * abs(want) + 1e-12
    g_in, g_out = d_in.cpu().numpy(), d_out.cpu().numpy()
    assert np.abs(g_in - h_in).max() <= EMB_ATOL
    assert np.abs(g_out - h_out).max() <= EMB_ATOL
    return g_in, g_out


@pytest.mark.parametrize("dim,k,b", [(64, 5, 65_536), (128, 5, 50_001), (256, 10, 9_999),
                                     (100, 3, 7_777), (4, 1, 513), (512, 2, 2_000),
                                     (1024, 60, 257), (768, 0, 1_000), (32, 60, 4_000)])
def test_sgns_step_mid_training_state(gs, oracle, dim, k, b):
    from paper_2407_15452_amd import inputs
    n = 5000
    w_in, w_out = inputs.random_tables(n, dim, seed=dim + k, scale=2.0 / dim ** 0.5)
    rng = np.random.default_rng(b)
    # skip-gram-like structure: runs of equal centres, power-law negatives
    c = np.repeat(rng.integers(0, n, b // 8 + 1), 8)[:b].astype(np.int32)
    o = rng.integers(0, n, b).astype(np.int32)
    neg = (n * rng.random((b, k)) ** 3).astype(np.int32)
    _sgns_case(gs, oracle, w_in, w_out, c, o, neg, 0.025)


def test_sgns_step_from_initial_state_workload0(gs, oracle, cfg0):
    """First batch of workload 0 from its initial tables (context table zero)."""
    from paper_2407_15452_amd import inputs
    wl, (off, nb), g = cfg0
    w_in, w_out = inputs.init_tables(wl.num_nodes, wl.dim, wl.init_seed)
    starts = _walk_inputs(wl, 500)
    walks = oracle.random_walk(off, nb, starts.numpy(), wl.walk_len, wl.walk_seed)
    c, o = oracle.make_pairs(walks, wl.window)
    c, o = c[:wl.batch_pairs], o[:wl.batch_pairs]
    nw = inputs.noise_weights(torch.as_tensor(off)).numpy()
    table = oracle.alias_build(np.array([0, wl.num_nodes], dtype=np.int32), nw)
    neg = oracle.sample_negatives(table, wl.num_nodes, c.size, wl.num_neg, wl.neg_seed)
    g_in, g_out = _sgns_case(gs, oracle, w_in, w_out, c, o, neg, 0.025)
    np.testing.assert_array_equal(g_in, w_in.numpy())      # closed form: no change at step one
    # rows the batch does not name are bit-unchanged
    named = np.zeros(wl.num_nodes, bool)
    named[o] = True
    named[neg.ravel()] = True
    assert (g_out[~named] == 0).all() and named.sum() < wl.num_nodes


def test_sgns_step_untouched_rows_and_empty_batch(gs, oracle):
    from paper_2407_15452_amd import inputs
    n, dim = 4000, 128
    w_in, w_out = inputs.random_tables(n, dim, seed=3, scale=0.2)
    rng = np.random.default_rng(0)
    b, k = 3000, 5
    c = rng.integers(0, n // 2, b).astype(np.int32)
    o = rng.integers(0, n // 2, b).astype(np.int32)
    neg = rng.integers(0, n // 2, (b, k)).astype(np.int32)
    g_in, g_out = _sgns_case(gs, oracle, w_in, w_out, c, o, neg, 0.05)
    np.testing.assert_array_equal(g_in[n // 2:], w_in.numpy()[n // 2:])
    np.testing.assert_array_equal(g_out[n // 2:], w_out.numpy()[n // 2:])
    d_in, d_out = w_in.to(DEV), w_out.to(DEV)
    e = torch.zeros(0, dtype=torch.int32, device=DEV)
    loss = gs.gs_sgns_step(d_in, d_out, e, e, torch.zeros((0, k), dtype=torch.int32, device=DEV), 0.1)
    assert float(loss.item()) == 0.0
    assert torch.equal(d_in.cpu(), w_in) and torch.equal(d_out.cpu(), w_out)


def test_sgns_step_argument_errors(gs):
    w = torch.zeros((10, 6), dtype=torch.float32, device=DEV)
    i = torch.zeros(4, dtype=torch.int32, device=DEV)
    n = torch.zeros((4, 2), dtype=torch.int32, device=DEV)
    with pytest.raises(gs.GsError):            # dim not a multiple of 4
        gs.gs_sgns_step(w, w.clone(), i, i, n, 0.1)
    w = torch.zeros((10, 8), dtype=torch.float32, device=DEV)
    with pytest.raises(gs.GsError) as ei:
        gs.gs_sgns_step(w, w.clone(), i, i, n, 0.1,
                        ws=torch.empty(256, dtype=torch.uint8, device=DEV))
    assert ei.value.status == gs.GS_EWORKSPACE


def test_epoch_of_workload0(gs, oracle, cfg0):
    """Whole pipeline on workload 0, one epoch, both sides from the same inputs."""
    from paper_2407_15452_amd import inputs
    wl, (off, nb), g = cfg0
    nw = wl.num_nodes * wl.walks_per_node
    starts = _walk_inputs(wl, nw)
    noise_w = inputs.noise_weights(torch.as_tensor(off))
    seg = np.array([0, wl.num_nodes], dtype=np.int32)
    # --- oracle side
    walks = oracle.random_walk(off, nb, starts.numpy(), wl.walk_len, wl.walk_seed)
    oc, oo = oracle.make_pairs(walks, wl.window)
    table = oracle.alias_build(seg, noise_w.numpy())
    oneg = oracle.sample_negatives(table, wl.num_nodes, oc.size, wl.num_neg, wl.neg_seed)
    # --- device side
    d_walks = gs.gs_random_walk(g, None, starts.to(DEV), wl.walk_len, wl.walk_seed)
    dc, do, n_pairs = gs.gs_make_pairs(d_walks, wl.window)
    noise = gs.gs_alias_build(_t(seg), noise_w.to(DEV))
    dneg = gs.gs_sample_negatives(noise, wl.num_nodes, n_pairs, wl.num_neg, wl.neg_seed)
    assert n_pairs == oc.size
    np.testing.assert_array_equal(dc.cpu().numpy(), oc)
    np.testing.assert_array_equal(do.cpu().numpy(), oo)
    np.testing.assert_array_equal(dneg.cpu().numpy(), oneg)

    w_in, w_out = inputs.init_tables(wl.num_nodes, wl.dim, wl.init_seed)
    h_in, h_out = w_in.numpy().copy(), w_out.numpy().copy()
    d_in, d_out = w_in.to(DEV), w_out.to(DEV)
    bsz = wl.batch_pairs
    nb_batches = (n_pairs + bsz - 1) // bsz
    assert nb_batches == 80          # 30,776 live walks x 170 pairs / 65,536
    ws = torch.empty(gs.gs_sgns_step_workspace_bytes(bsz, wl.num_nodes, wl.num_neg, wl.dim), dtype=torch.uint8,
                     device=DEV)
    losses = torch.zeros(nb_batches, dtype=torch.float64, device=DEV)
    o_loss = 0.0
    for b in range(nb_batches):
        lo, hi = b * bsz, min(n_pairs, (b + 1) * bsz)
        lr = inputs.learning_rate(wl, b, nb_batches)
        gs.gs_sgns_step(d_in, d_out, dc[lo:hi], do[lo:hi], dneg[lo:hi], lr,
                        loss_out=losses[b:b + 1], ws=ws)
        o_loss += oracle.sgns_step(h_in, h_out, oc[lo:hi], oo[lo:hi], oneg[lo:hi], lr)
    torch.cuda.synchronize()
    d_loss = float(losses.sum().item())
    assert abs(d_loss - o_loss) / abs(o_loss) <= 1e-3
    for got, want in ((d_in.cpu().numpy(), h_in), (d_out.cpu().numpy(), h_out)):
        na, nb_ = np.linalg.norm(got, axis=1), np.linalg.norm(want, axis=1)
        live = (na > 0) | (nb_ > 0)
        cos = (got[live] * want[live]).sum(1) / np.maximum(na[live] * nb_[live], 1e-30)
        assert cos.mean() >= 0.999


# ----------------------------------------------------------------------------- SGNS, bf16 tables
def _bf16_bits(t):
    return t.view(torch.int16).cpu().numpy().view(np.uint16).copy()


@pytest.mark.parametrize("dim,k,b", [(256, 10, 30_011), (128, 5, 50_001), (64, 5, 9_999),
                                     (192, 3, 5_000), (8, 1, 513), (1024, 4, 1_000),
                                     (512, 60, 300)])
@pytest.mark.parametrize("fmt", ["bf16", "f16"])
def test_sgns_step_bf16_tables(gs, oracle, dim, k, b, fmt):
    """16-bit storage (bfloat16, IEEE binary16), one rounding per written element.

    Both sides add a row's terms exactly and round once, but the terms themselves come from
    fp32 arithmetic on the GPU (dot products, sigmoid), so a sum that lands on a rounding
    boundary of the 16-bit format may round the other way: all elements must agree to within
    one step of the format (or the fp32 bound where the sum cancels), and all but 1e-4
    (bfloat16) or 1e-3 (binary16) of them must be bit-identical."""
    from paper_2407_15452_amd import inputs
    n = 5000
    f_in, f_out = inputs.random_tables(n, dim, seed=dim + k, scale=2.0 / dim ** 0.5)
    tdt, code = (torch.bfloat16, oracle.BF16) if fmt == "bf16" else (torch.float16, oracle.F16)
    b_in, b_out = f_in.to(tdt), f_out.to(tdt)
    rng = np.random.default_rng(b)
    c = np.repeat(rng.integers(0, n, b // 8 + 1), 8)[:b].astype(np.int32)
    o = rng.integers(0, n, b).astype(np.int32)
    neg = (n * rng.random((b, k)) ** 3).astype(np.int32)      # hub rows get thousands of terms
    h_in, h_out = _bf16_bits(b_in), _bf16_bits(b_out)
    before_in, before_out = h_in.copy(), h_out.copy()
    want = oracle.sgns_step(h_in, h_out, c, o, neg, 0.025, dtype=code)
    d_in, d_out = b_in.to(DEV), b_out.to(DEV)
    loss = gs.gs_sgns_step(d_in, d_out, _t(c), _t(o), _t(neg), 0.025)
    torch.cuda.synchronize()
    assert abs(float(loss.item()) - want) <= LOSS_RTOL * abs(want)
    for got_t, want_bits, before in ((d_in, h_in, before_in), (d_out, h_out, before_out)):
        got_bits = _bf16_bits(got_t)
        touched = want_bits != before
        assert touched.any()
        assert_half_close(got_bits, want_bits, fmt)
        # rows the batch does not name keep their bits
        named = np.zeros(n, bool)
        named[c] = True
        named[o] = True
        named[neg.ravel()] = True
        np.testing.assert_array_equal(got_bits[~named], before[~named])


def test_sgns_step_bf16_rejects_odd_dims(gs):
    w = torch.zeros((10, 12), dtype=torch.bfloat16, device=DEV)
    i = torch.zeros(4, dtype=torch.int32, device=DEV)
    with pytest.raises(gs.GsError):
        gs.gs_sgns_step(w, w.clone(), i, i, torch.zeros((4, 2), dtype=torch.int32, device=DEV), 0.1)


# ----------------------------------------------------------------------------- workloads 3 and 4, scaled down
def _pipeline_parity(gs, oracle, wl, num_walks, loss_rtol=LOSS_RTOL):
    """Whole path on a (scaled) workload: every stage against the oracle."""
    from paper_2407_15452_amd import inputs
    src, dst, w = inputs.edge_list(wl, "cpu")
    flags = oracle.DROP_SELF_LOOPS | oracle.DEDUPE | (0 if wl.directed else oracle.SYMMETRIZE)
    hw = None if w is None else w.numpy()
    off, nb, wo = oracle.csr_build(src.numpy(), dst.numpy(), hw, wl.num_nodes, flags, wl.offset_bits)
    g = gs.gs_csr_build(src.to(DEV), dst.to(DEV), None if w is None else w.to(DEV), wl.num_nodes,
                        flags, wl.offset_bits)
    np.testing.assert_array_equal(g.offsets.cpu().numpy(), off)
    np.testing.assert_array_equal(g.nbrs.cpu().numpy(), nb)
    table = d_table = None
    if wl.weighted:
        np.testing.assert_array_equal(g.weights.cpu().numpy(), wo)
        table = oracle.alias_build(off, wo)
        d_table = gs.gs_alias_build(g.offsets, g.weights)
        np.testing.assert_array_equal(d_table.prob.cpu().numpy(), table[0])
        np.testing.assert_array_equal(d_table.alias.cpu().numpy(), table[1])
    starts = inputs.walk_starts(wl.num_nodes, 0, num_walks)
    if wl.node2vec:
        walks = oracle.node2vec_walk(off, nb, starts.numpy(), wl.walk_len, wl.p, wl.q, wl.walk_seed,
                                     alias=table)
        d_walks = gs.gs_node2vec_walk(g, d_table, starts.to(DEV), wl.walk_len, wl.p, wl.q,
                                      wl.walk_seed)
    else:
        walks = oracle.random_walk(off, nb, starts.numpy(), wl.walk_len, wl.walk_seed, alias=table)
        d_walks = gs.gs_random_walk(g, d_table, starts.to(DEV), wl.walk_len, wl.walk_seed)
    np.testing.assert_array_equal(d_walks.cpu().numpy(), walks)
    oc, oo = oracle.make_pairs(walks, wl.window)
    dc, do, n_pairs = gs.gs_make_pairs(d_walks, wl.window)
    np.testing.assert_array_equal(dc.cpu().numpy(), oc)
    np.testing.assert_array_equal(do.cpu().numpy(), oo)
    noise_w = inputs.noise_weights(torch.as_tensor(off))
    seg = np.array([0, wl.num_nodes], dtype=np.int64)
    noise_t = oracle.alias_build(seg, noise_w.numpy())
    noise = gs.gs_alias_build(_t(seg), noise_w.to(DEV))
    b = min(n_pairs, 40_000)
    oneg = oracle.sample_negatives(noise_t, wl.num_nodes, b, wl.num_neg, wl.neg_seed)
    dneg = gs.gs_sample_negatives(noise, wl.num_nodes, b, wl.num_neg, wl.neg_seed)
    np.testing.assert_array_equal(dneg.cpu().numpy(), oneg)
    f_in, f_out = inputs.random_tables(wl.num_nodes, wl.dim, seed=9, scale=2.0 / wl.dim ** 0.5)
    if wl.dtype == "bf16":
        b_in, b_out = f_in.to(torch.bfloat16), f_out.to(torch.bfloat16)
        h_in, h_out = _bf16_bits(b_in), _bf16_bits(b_out)
        want = oracle.sgns_step(h_in, h_out, oc[:b], oo[:b], oneg, 0.025, dtype=oracle.BF16)
        d_in, d_out = b_in.to(DEV), b_out.to(DEV)
        loss = gs.gs_sgns_step(d_in, d_out, dc[:b], do[:b], dneg, 0.025)
        assert abs(float(loss.item()) - want) <= loss_rtol * abs(want)
        for got_t, want_bits in ((d_in, h_in), (d_out, h_out)):
            assert_half_close(_bf16_bits(got_t), want_bits, "bf16")
    else:
        _sgns_case(gs, oracle, f_in, f_out, oc[:b], oo[:b], oneg, 0.025)
    return walks


def test_workload3_scaled_weighted_bipartite_bf16(gs, oracle):
    from paper_2407_15452_amd import inputs
    wl = inputs.WORKLOADS[3].scaled(1e-3)
    assert wl.weighted and wl.dtype == "bf16" and wl.num_neg == 10 and wl.dim == 256
    walks = _pipeline_parity(gs, oracle, wl, 3000)
    # bipartite: users and items alternate along every walk
    nu = wl.num_users
    live = walks[:, 1] >= 0
    assert live.any()
    side = walks[live][:, :2] >= nu
    assert (side[:, 0] != side[:, 1]).all()


def test_workload4_scaled_directed_int64_offsets(gs, oracle):
    from paper_2407_15452_amd import inputs
    wl = inputs.WORKLOADS[4].scaled(1e-3)
    assert wl.directed and wl.offset_bits == 64
    walks = _pipeline_parity(gs, oracle, wl, 20_000)
    assert (walks == -1).any()                 # directed R-MAT: walks do end at sinks


def test_workload2_scaled_node2vec(gs, oracle):
    from paper_2407_15452_amd import inputs
    wl = inputs.WORKLOADS[2].scaled(5e-3)
    _pipeline_parity(gs, oracle, wl, 2_000)


# ----------------------------------------------------------------------------- alias, long single segment
@pytest.mark.parametrize("kind", ["one_giant", "equal", "two_level", "lognormal", "mostly_zero"])
def test_alias_build_long_segment_shapes(gs, oracle, kind):
    """The workgroup construction of one long segment against the oracle's
    sequential one, on weight shapes that stress its serial and parallel parts."""
    rng = np.random.default_rng(42)
    n = 50_003
    if kind == "one_giant":                     # one entry absorbs all the others, one at a time
        w = np.full(n, 1e-3, dtype=np.float32)
        w[n // 3] = 1e6
    elif kind == "equal":
        w = np.full(n, 0.75, dtype=np.float32)
    elif kind == "two_level":                   # half just below, half just above the mean
        w = np.where(np.arange(n) % 2 == 0, 0.9, 1.1).astype(np.float32)
    elif kind == "lognormal":
        w = rng.lognormal(0, 2.5, n).astype(np.float32)
    else:
        w = np.zeros(n, dtype=np.float32)
        w[rng.choice(n, 300, replace=False)] = rng.random(300).astype(np.float32) + 0.1
    seg = np.array([0, n], dtype=np.int64)
    prob, alias = oracle.alias_build(seg, w)
    a = gs.gs_alias_build(_t(seg), _t(w))
    np.testing.assert_array_equal(a.alias.cpu().numpy(), alias)
    np.testing.assert_array_equal(a.prob.cpu().numpy(), prob)


def test_packed_alias_layout_changes_nothing(gs, oracle, cfg0):
    """Samplers read the interleaved table when it is given; results are the same."""
    wl, (off, nb), g = cfg0
    rng = np.random.default_rng(3)
    w = rng.lognormal(0, 1, nb.size).astype(np.float32)
    plain = gs.gs_alias_build(g.offsets, _t(w), pack=False)
    packed = gs.gs_alias_build(g.offsets, _t(w), pack=True)
    assert plain.packed is None and packed.packed is not None
    bits = packed.packed.cpu().numpy().view(np.uint64)
    np.testing.assert_array_equal((bits & 0xFFFFFFFF).astype(np.uint32),
                                  packed.prob.cpu().numpy().view(np.uint32))
    np.testing.assert_array_equal((bits >> 32).astype(np.int32), packed.alias.cpu().numpy())
    starts = _walk_inputs(wl, 5000).to(DEV)
    a = gs.gs_random_walk(g, plain, starts, 20, 7)
    b = gs.gs_random_walk(g, packed, starts, 20, 7)
    assert torch.equal(a, b)
    a = gs.gs_node2vec_walk(g, plain, starts, 20, 0.5, 2.0, 7)
    b = gs.gs_node2vec_walk(g, packed, starts, 20, 0.5, 2.0, 7)
    assert torch.equal(a, b)
    nw = _t(np.arange(1, wl.num_nodes + 1, dtype=np.float32))
    seg = _t(np.array([0, wl.num_nodes], dtype=np.int64))
    n_plain = gs.gs_alias_build(seg, nw, pack=False)
    n_packed = gs.gs_alias_build(seg, nw, pack=True)
    a = gs.gs_sample_negatives(n_plain, wl.num_nodes, 20_000, 5, 11)
    b = gs.gs_sample_negatives(n_packed, wl.num_nodes, 20_000, 5, 11)
    assert torch.equal(a, b)


# ----------------------------------------------------------------------------- SGD with momentum
@pytest.mark.parametrize("dim,k,b,dtype", [(128, 5, 50_001, "f32"), (64, 3, 7_777, "f32"),
                                           (256, 10, 9_999, "bf16"), (128, 5, 9_999, "f16")])
def test_sgns_momentum_step(gs, oracle, dim, k, b, dtype):
    """Three consecutive mult / put / mult_add iterations against the oracle."""
    from paper_2407_15452_amd import inputs
    n = 5000
    f_in, f_out = inputs.random_tables(n, dim, seed=dim + k, scale=2.0 / dim ** 0.5)
    m_a, m_b = inputs.random_tables(n, dim, seed=dim + k + 1, scale=0.01)
    tdt = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}[dtype]
    half = dtype != "f32"                                   # a 16-bit storage format
    ulp = 2.0 ** -7 if dtype == "bf16" else 2.0 ** -10       # relative size of one step
    tabs = [t.to(tdt) for t in (f_in, f_out, m_a, m_b)]
    host = [_bf16_bits(t) if half else t.numpy().copy() for t in tabs]
    dev = [t.to(DEV) for t in tabs]
    odt = {"bf16": oracle.BF16, "f16": oracle.F16, "f32": oracle.F32}[dtype]
    rng = np.random.default_rng(b)
    lr, mu = 0.025, 0.9
    for it in range(3):
        c = np.repeat(rng.integers(0, n, b // 8 + 1), 8)[:b].astype(np.int32)
        o = rng.integers(0, n, b).astype(np.int32)
        neg = (n * rng.random((b, k)) ** 3).astype(np.int32)
        old_model = [h.copy() for h in host[:2]]
        want = oracle.sgns_momentum_step(*host, c, o, neg, lr, mu, dtype=odt)
        loss = gs.gs_sgns_momentum_step(*dev, _t(c), _t(o), _t(neg), lr, mu)
        torch.cuda.synchronize()
        assert abs(float(loss.item()) - want) <= LOSS_RTOL * abs(want)
        if dtype == "f16":
            f32 = lambda bits: bits.view(np.float16).astype(np.float32)  # noqa: E731
        else:
            f32 = lambda bits: (bits.astype(np.uint32) << 16).view(np.float32)  # noqa: E731
        for which, (d_t, h_t) in enumerate(zip(dev, host)):
            if half and which >= 2:
                # momentum tables: one rounding after the fp32 / fp64 gradient sum
                assert_half_close(_bf16_bits(d_t), h_t, dtype)
            elif half:
                # model tables: a momentum entry that rounded the other way moves the model by
                # lr times a whole bf16 step of the momentum, so the mult_add is checked against
                # the momentum the GPU itself holds: w' = bf16(w - lr * m')
                got = _bf16_bits(d_t)
                m_new = f32(_bf16_bits(dev[which + 2]))
                w_old = f32(old_model[which])
                expect = w_old - np.float32(lr) * m_new
                # within one bf16 step of the exact value (2^-7 relative to the larger operand)
                scale = np.maximum(np.abs(w_old), np.abs(np.float32(lr) * m_new))
                # (binary16 results below 6e-5 are subnormal: steps of 6e-8 there)
                excess = np.abs(f32(got) - expect) - (ulp * scale + 6e-8)
                assert excess.max() <= 0, float(excess.max())
            else:
                # (momentum entries are unscaled gradient sums: magnitudes of 50 in the hub rows
                # of this batch, where the bound is 16 fp32 spacings of the value)
                assert_emb_close(d_t.cpu().numpy(), h_t)
        if half:                                            # next iteration from a common state
            for d_t, h_t in zip(dev, host):
                d_t.copy_(torch.from_numpy(h_t.view(np.int16)).view(tdt))


def test_sgns_momentum_step_argument_errors(gs):
    w = [torch.zeros((10, 8), dtype=torch.float32, device=DEV) for _ in range(4)]
    i = torch.zeros(4, dtype=torch.int32, device=DEV)
    n = torch.zeros((4, 2), dtype=torch.int32, device=DEV)
    with pytest.raises(gs.GsError):            # momentum table aliasing a model table
        gs.gs_sgns_momentum_step(w[0], w[1], w[0], w[3], i, i, n, 0.1, 0.9)
    loss = gs.gs_sgns_momentum_step(*w, i, i, n, 0.1, 0.9)
    assert float(loss.item()) == pytest.approx(4 * 3 * np.log(2.0))


# ----------------------------------------------------------------------------- Adam
@pytest.mark.parametrize("dim,k,b,eps", [(128, 5, 50_001, 1e-8), (64, 3, 7_777, 1e-8),
                                         (256, 10, 9_999, 1e-4), (320, 2, 4_096, 1e-8)])
def test_sgns_adam_step(gs, oracle, dim, k, b, eps):
    """Three consecutive Adam iterations (dense decay, sparse put, dense apply) against the
    oracle.  Both moments are compared element by element.  The model is compared (a) with
    the apply formula evaluated in fp64 from the moments the GPU itself holds, on every
    element, and (b) with the oracle wherever the denominator sqrt(v)/sqrt(1-beta2^t)+eps is
    at least 1e-3: below that the update lr*m/denominator magnifies the fp32 summation
    noise of a gradient that cancels to almost zero (an element whose gradient is 1e-9 on
    one side and -1e-9 on the other moves by +lr or -lr), which no summation order fixes."""
    from paper_2407_15452_amd import inputs
    n = 5000
    f_in, f_out = inputs.random_tables(n, dim, seed=dim + k, scale=2.0 / dim ** 0.5)
    zeros = [torch.zeros((n, dim), dtype=torch.float32) for _ in range(4)]
    host = [t.numpy().copy() for t in (f_in, f_out, *zeros)]
    dev = [t.to(DEV) for t in (f_in, f_out, *zeros)]
    rng = np.random.default_rng(b)
    lr, b1, b2 = 0.01, 0.9, 0.999
    for it in range(1, 4):
        c = np.repeat(rng.integers(0, n, b // 8 + 1), 8)[:b].astype(np.int32)
        o = rng.integers(0, n, b).astype(np.int32)
        neg = (n * rng.random((b, k)) ** 3).astype(np.int32)
        old_model = [h.copy() for h in host[:2]]
        want = oracle.sgns_adam_step(*host, c, o, neg, lr, b1, b2, eps, it)
        loss = gs.gs_sgns_adam_step(*dev, _t(c), _t(o), _t(neg), lr, b1, b2, eps, it)
        torch.cuda.synchronize()
        assert abs(float(loss.item()) - want) <= LOSS_RTOL * abs(want)
        got = [d.cpu().numpy() for d in dev]
        for which in (2, 3, 4, 5):                       # m_in, m_out, v_in, v_out
            assert (np.abs(got[which] - host[which]) <= 1e-6 + 1e-5 * np.abs(host[which])).all()
        step = np.float64(np.float32(lr)) / (1.0 - np.float64(np.float32(b1)) ** it)
        root = np.sqrt(1.0 - np.float64(np.float32(b2)) ** it)
        for which in (0, 1):
            m, v = got[which + 2].astype(np.float64), got[which + 4].astype(np.float64)
            denom = np.sqrt(v) / root + np.float64(np.float32(eps))
            expect = old_model[which].astype(np.float64) - step * m / np.where(denom > 0, denom, 1.0)
            assert np.abs(got[which] - expect).max() <= 1e-6
            safe = (np.sqrt(host[which + 4].astype(np.float64)) / root + eps) >= 1e-3
            assert safe.mean() > 0.5 if which == 1 else True
            assert np.abs(got[which] - host[which])[safe].max() <= EMB_ATOL
            assert np.abs(got[which] - host[which]).max() <= 2.0 * step + EMB_ATOL
            untouched = host[which + 4].max(axis=1) == 0   # rows no batch has named yet
            np.testing.assert_array_equal(got[which][untouched], old_model[which][untouched])
        for d_t, h_t in zip(dev, host):                      # next iteration from a common state
            d_t.copy_(torch.from_numpy(h_t))


def test_sgns_adam_step_argument_errors(gs):
    w = [torch.zeros((10, 8), dtype=torch.float32, device=DEV) for _ in range(6)]
    i = torch.zeros(4, dtype=torch.int32, device=DEV)
    n = torch.zeros((4, 2), dtype=torch.int32, device=DEV)
    with pytest.raises(gs.GsError):            # a moment table aliasing another table
        gs.gs_sgns_adam_step(w[0], w[1], w[2], w[3], w[2], w[5], i, i, n, 0.1, 0.9, 0.999, 1e-8, 1)
    with pytest.raises(gs.GsError):            # iteration numbers start at 1
        gs.gs_sgns_adam_step(*w, i, i, n, 0.1, 0.9, 0.999, 1e-8, 0)
    with pytest.raises(gs.GsError):
        gs.gs_sgns_adam_step(*w, i, i, n, 0.1, 1.0, 0.999, 1e-8, 1)
    with pytest.raises(TypeError):
        gs.gs_sgns_adam_step(w[0].to(torch.bfloat16), *w[1:], i, i, n, 0.1, 0.9, 0.999, 1e-8, 1)
    loss = gs.gs_sgns_adam_step(*w, i, i, n, 0.1, 0.9, 0.999, 1e-8, 1)
    assert float(loss.item()) == pytest.approx(4 * 3 * np.log(2.0))


# ----------------------------------------------------------------------------- fused negatives
@pytest.mark.parametrize("dim,k,b,dtype,weighted,pack", [(128, 5, 50_001, "f32", True, True),
                                                         (64, 3, 7_777, "f32", True, False),
                                                         (64, 5, 65_536, "f32", False, False),
                                                         (256, 10, 9_999, "bf16", True, True),
                                                         (128, 0, 1_000, "f32", True, True)])
def test_sgns_step_fused_draws_the_same_negatives(gs, oracle, cfg0, dim, k, b, dtype, weighted, pack):
    """The fused call against the oracle's sample_negatives + sgns_step, two consecutive
    batches with a pair index base beyond 32 bits."""
    from paper_2407_15452_amd import inputs
    wl, (off, nb), g = cfg0
    n = wl.num_nodes
    noise_h = noise_d = None
    if weighted:
        nw = inputs.noise_weights(torch.as_tensor(off)).numpy()
        seg = np.array([0, n], dtype=np.int32)
        noise_h = oracle.alias_build(seg, nw)
        noise_d = gs.gs_alias_build(_t(seg), _t(nw), pack=pack)
    f_in, f_out = inputs.random_tables(n, dim, seed=dim + k, scale=2.0 / dim ** 0.5)
    rng = np.random.default_rng(b)
    if dtype == "bf16":
        d_in, d_out = f_in.to(torch.bfloat16).to(DEV), f_out.to(torch.bfloat16).to(DEV)
        h_in, h_out = _bf16_bits(d_in).copy(), _bf16_bits(d_out).copy()
        code = oracle.BF16
    else:
        d_in, d_out = f_in.to(DEV), f_out.to(DEV)
        h_in, h_out = f_in.numpy().copy(), f_out.numpy().copy()
        code = oracle.F32
    base = (1 << 34) + 11
    for it in range(2):
        c = np.repeat(rng.integers(0, n, b // 8 + 1), 8)[:b].astype(np.int32)
        o = rng.integers(0, n, b).astype(np.int32)
        neg = oracle.sample_negatives(noise_h, n, b, k, seed=99, pair_index_base=base + it * b)
        if k == 0:
            neg = np.zeros((b, 0), dtype=np.int32)
        want = oracle.sgns_step(h_in, h_out, c, o, neg, 0.01, dtype=code)
        loss = gs.gs_sgns_step_fused(d_in, d_out, _t(c), _t(o), noise_d, k, 99, 0.01,
                                     pair_index_base=base + it * b)
        torch.cuda.synchronize()
        assert abs(float(loss.item()) - want) <= LOSS_RTOL * abs(want)
        if dtype == "bf16":
            for d_t, h_t in ((d_in, h_in), (d_out, h_out)):
                assert_half_close(_bf16_bits(d_t), h_t, "bf16")
                d_t.copy_(torch.from_numpy(h_t.view(np.int16)).view(torch.bfloat16))
        else:
            assert np.abs(d_in.cpu().numpy() - h_in).max() <= EMB_ATOL
            assert np.abs(d_out.cpu().numpy() - h_out).max() <= EMB_ATOL


def test_sgns_step_fused_argument_errors(gs):
    w = [torch.zeros((10, 8), dtype=torch.float32, device=DEV) for _ in range(2)]
    i = torch.zeros(4, dtype=torch.int32, device=DEV)
    small = torch.empty(256, dtype=torch.uint8, device=DEV)
    with pytest.raises(gs.GsError):
        gs.gs_sgns_step_fused(w[0], w[1], i, i, None, 2, 1, 0.1, ws=small)
    with pytest.raises(gs.GsError):
        gs.gs_sgns_step_fused(w[0], w[1], i, i, None, 61, 1, 0.1)
    loss = gs.gs_sgns_step_fused(w[0], w[1], i, i, None, 2, 1, 0.1)
    assert float(loss.item()) == pytest.approx(4 * 3 * np.log(2.0))


# ----------------------------------------------------------------------------- graph capture
def test_step_replays_from_a_captured_graph(gs, oracle, cfg0):
    """gs_sample_negatives + gs_sgns_step captured once into a HIP graph (the library clears
    its scratch with fill kernels, allocates nothing and never synchronises) and replayed
    on fresh batches, with eager work and synchronisation between the replays; every
    replay is checked against the oracle."""
    from paper_2407_15452_amd import inputs
    wl, (off, nb), g = cfg0
    n, d, k, b = wl.num_nodes, wl.dim, wl.num_neg, 8_192
    nw = inputs.noise_weights(torch.as_tensor(off)).numpy()
    seg = np.array([0, n], dtype=np.int32)
    noise_h = oracle.alias_build(seg, nw)
    noise_d = gs.gs_alias_build(_t(seg), _t(nw))
    f_in, f_out = inputs.random_tables(n, d, seed=3, scale=0.25)
    d_in, d_out = f_in.to(DEV), f_out.to(DEV)
    h_in, h_out = f_in.numpy().copy(), f_out.numpy().copy()
    c_buf = torch.zeros(b, dtype=torch.int32, device=DEV)
    o_buf = torch.zeros(b, dtype=torch.int32, device=DEV)
    negs = torch.zeros((b, k), dtype=torch.int32, device=DEV)
    loss = torch.zeros(1, dtype=torch.float64, device=DEV)
    ws = torch.empty(gs.gs_sgns_step_workspace_bytes(b, n, k, d), dtype=torch.uint8, device=DEV)
    rng = np.random.default_rng(4)

    def body():
        gs.gs_sample_negatives(noise_d, n, b, k, 17, pair_index_base=5, out=negs)
        gs.gs_sgns_step(d_in, d_out, c_buf, o_buf, negs, 0.01, loss_out=loss, ws=ws)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        body()                                   # warm-up outside capture (on zeros: ids 0)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    d_in.copy_(f_in); d_out.copy_(f_out)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        body()
    d_in.copy_(f_in); d_out.copy_(f_out)         # capture does not run the kernels; start clean
    h_neg = oracle.sample_negatives(noise_h, n, b, k, 17, pair_index_base=5)
    for it in range(4):
        c = np.repeat(rng.integers(0, n, b // 8), 8).astype(np.int32)
        o = rng.integers(0, n, b).astype(np.int32)
        c_buf.copy_(_t(c)); o_buf.copy_(_t(o))
        graph.replay()
        torch.cuda.synchronize()
        want = oracle.sgns_step(h_in, h_out, c, o, h_neg, 0.01)
        assert abs(float(loss.item()) - want) <= LOSS_RTOL * abs(want)
        np.testing.assert_array_equal(negs.cpu().numpy(), h_neg)
        assert np.abs(d_in.cpu().numpy() - h_in).max() <= EMB_ATOL * (it + 1)
        assert np.abs(d_out.cpu().numpy() - h_out).max() <= EMB_ATOL * (it + 1)
        # eager work of the program's own between the replays
        _ = (d_in * 2).sum().item()


@pytest.mark.parametrize("bits", [32, 64])
def test_alias_build_rows_of_hub_nodes(gs, oracle, bits):
    """Per-row tables of a graph whose hub rows are long enough for the workgroup kernel
    (>= 8192 entries), next to rows just below the threshold, short rows and empty rows."""
    rng = np.random.default_rng(bits)
    lens = np.concatenate([[20_000, 0, 8_192, 8_191, 1, 0, 50_000, 9_000],
                           rng.integers(0, 40, 3_000), [12_345]]).astype(np.int64)
    off = np.concatenate([[0], np.cumsum(lens)])
    total = int(off[-1])
    w = rng.lognormal(0, 2.0, total).astype(np.float32)
    w[rng.random(total) < 0.05] = 0
    w[off[6]:off[6] + 10] = 1e6                              # a few very heavy entries in a hub row
    off = off.astype(np.int64 if bits == 64 else np.int32)
    prob, alias = oracle.alias_build(off, w)
    a = gs.gs_alias_build(_t(off), _t(w))
    np.testing.assert_array_equal(a.alias.cpu().numpy(), alias)
    np.testing.assert_array_equal(a.prob.cpu().numpy(), prob)


def test_sgns_step_reports_ids_that_are_not_rows(gs):
    """Ids outside [0, num_nodes) cannot be seen by the host: the kernels treat them as row 0
    (no access outside the tables) and the loss comes back as NaN; a clean call afterwards
    with the same workspace reports a finite loss again."""
    n, d, b, k = 1000, 64, 4096, 3
    rng = np.random.default_rng(0)
    w_in = torch.zeros((n, d), dtype=torch.float32, device=DEV)
    w_out = torch.zeros((n, d), dtype=torch.float32, device=DEV)
    c = rng.integers(0, n, b).astype(np.int32)
    o = rng.integers(0, n, b).astype(np.int32)
    neg = rng.integers(0, n, (b, k)).astype(np.int32)
    ws = torch.empty(gs.gs_sgns_step_workspace_bytes(b, n, k, d), dtype=torch.uint8, device=DEV)
    for which in range(3):
        bad = [c.copy(), o.copy(), neg.copy()]
        bad[which].reshape(-1)[17] = n if which != 1 else -1
        loss = gs.gs_sgns_step(w_in, w_out, _t(bad[0]), _t(bad[1]), _t(bad[2]), 0.01, ws=ws)
        assert np.isnan(float(loss.item()))
    loss = gs.gs_sgns_step(w_in, w_out, _t(c), _t(o), _t(neg), 0.01, ws=ws)
    assert np.isfinite(float(loss.item()))
    with pytest.raises(gs.GsError):            # one table on both sides
        gs.gs_sgns_step(w_in, w_in, _t(c), _t(o), _t(neg), 0.01, ws=ws)


def test_walks_stop_at_neighbour_ids_that_are_not_nodes(gs):
    """A hand-made CSR with entries outside [0, num_nodes): the walkers end the walk there
    (-1 from then on) instead of reading past the offsets."""
    n = 6
    off = torch.tensor([0, 2, 3, 4, 4, 5, 6], dtype=torch.int32, device=DEV)
    nb = torch.tensor([1, 2, 6, 0, 1_000_000, -7], dtype=torch.int32, device=DEV)   # rows 1, 4, 5 are bad
    g = gs.Csr(off, nb)
    starts = torch.arange(n, dtype=torch.int32, device=DEV).repeat(50)
    for walks in (gs.gs_random_walk(g, None, starts, 12, seed=3),
                  gs.gs_node2vec_walk(g, None, starts, 12, 0.5, 2.0, seed=3)):
        w = walks.cpu().numpy()
        assert ((w >= -1) & (w < n)).all()
        assert (w[:, 0] == starts.cpu().numpy()).all()
        dead = w == -1
        assert (dead[:, 1:] >= dead[:, :-1]).all()             # -1 only as a suffix
        assert (w[starts.cpu().numpy() == 1][:, 1] == -1).all()


@pytest.mark.parametrize("fmt", ["f32", "bf16"])
def test_sgns_step_same_bits_every_run(gs, fmt):
    """The same call on the same inputs gives the same bits: the row sums are exact integer
    sums, so neither the arrival order of a row's terms nor the way a long row is split
    matters.  Skewed batch (hub rows with tens of thousands of terms, runs of equal centres,
    hub centres with hundreds of runs), five runs, tables and loss compared bit by bit."""
    from paper_2407_15452_amd import inputs
    n, dim, b, k = 20_000, 128, 300_000, 5
    f_in, f_out = inputs.random_tables(n, dim, seed=77, scale=0.2)
    tdt = torch.float32 if fmt == "f32" else torch.bfloat16
    rng = np.random.default_rng(5)
    c = np.repeat((n * rng.random(b // 6 + 1) ** 4).astype(np.int32), 6)[:b]
    o = rng.integers(0, n, b).astype(np.int32)
    neg = (n * rng.random((b, k)) ** 4).astype(np.int32)
    dc, do, dn = _t(c), _t(o), _t(neg)
    results = []
    for run in range(5):
        d_in, d_out = f_in.to(tdt).to(DEV), f_out.to(tdt).to(DEV)
        loss = gs.gs_sgns_step(d_in, d_out, dc, do, dn, 0.025)
        torch.cuda.synchronize()
        results.append((d_in.view(torch.int16 if fmt == "bf16" else torch.int32).cpu(),
                        d_out.view(torch.int16 if fmt == "bf16" else torch.int32).cpu(),
                        loss.cpu().view(torch.int64)))
    for r in results[1:]:
        for x, y in zip(results[0], r):
            assert torch.equal(x, y)


@pytest.mark.parametrize("fmt", ["f32", "bf16"])
@pytest.mark.parametrize("b,k", [(1, 5), (37, 0), (2_048, 5), (9_000, 2)])
def test_sgns_step_small_batch_on_large_graph(gs, oracle, b, k, fmt):
    """The paper's own regime (Sec. 4: batches of 512 to 2048 source nodes on graphs of 10^8
    vertices): the batch names a tiny part of the rows, and nothing in the step has the size of
    the graph (two launches for these sizes; counters over the keys of a larger batch are in
    test_gpu_step_routes.py).  Hub rows with thousands of terms, runs of equal centres, centres
    that are also contexts; rows the batch does not name keep their bits."""
    from paper_2407_15452_amd import inputs
    n, dim = 400_000, 64
    f_in, f_out = inputs.random_tables(n, dim, seed=b + k, scale=0.25)
    rng = np.random.default_rng(b * 31 + k)
    c = np.repeat((n * rng.random(b // 5 + 1) ** 2).astype(np.int32), 5)[:b]
    o = rng.integers(0, n, b).astype(np.int32)
    o[::3] = c[::3]
    neg = (n * rng.random((b, k)) ** 6).astype(np.int32)          # a few rows take most draws
    if fmt == "f32":
        g_in, g_out = _sgns_case(gs, oracle, f_in, f_out, c, o, neg, 0.025)
        named = np.zeros(n, bool)
        named[c] = named[o] = True
        named[neg.ravel()] = True
        np.testing.assert_array_equal(g_in[~named], f_in.numpy()[~named])
        np.testing.assert_array_equal(g_out[~named], f_out.numpy()[~named])
    else:
        b_in, b_out = f_in.to(torch.bfloat16), f_out.to(torch.bfloat16)
        h_in, h_out = _bf16_bits(b_in), _bf16_bits(b_out)
        want = oracle.sgns_step(h_in, h_out, c, o, neg, 0.025, dtype=oracle.BF16)
        d_in, d_out = b_in.to(DEV), b_out.to(DEV)
        loss = gs.gs_sgns_step(d_in, d_out, _t(c), _t(o), _t(neg).reshape(b, k), 0.025)
        torch.cuda.synchronize()
        assert abs(float(loss.item()) - want) <= LOSS_RTOL * abs(want)
        # few elements are touched at all: one that rounds the other way is a large fraction
        assert_half_close(_bf16_bits(d_in), h_in, "bf16", flip_fraction=1e-3)
        assert_half_close(_bf16_bits(d_out), h_out, "bf16", flip_fraction=1e-3)


# ----------------------------------------------------------------------------- pairs made inside the step
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("walk_len,window,k", [(20, 5, 5), (7, 9, 3), (33, 2, 0)])
def test_sgns_step_from_walks(gs, oracle, walk_len, window, k, dtype):
    """gs_pair_offsets + gs_sgns_step_from_walks against the oracle's make_pairs +
    sample_negatives + sgns_step on the same walks: a directed graph with sinks (walks of every
    length, some without any pair), batches cut at arbitrary pair indices (inside walks, across
    several walks, the ragged last one), pair numbering continued over the batches."""
    from paper_2407_15452_amd import inputs
    n, dim = 3000, 64
    rng = np.random.default_rng(walk_len * 100 + window)
    src = rng.integers(0, n, 9000).astype(np.int32)
    dst = rng.integers(0, n, 9000).astype(np.int32)
    src[dst % 5 == 0] = dst[dst % 5 == 0]                # a fifth of the nodes only receive edges
    flags = oracle.DROP_SELF_LOOPS | oracle.DEDUPE
    off, nb, _ = oracle.csr_build(src, dst, None, n, flags)
    g = gs.gs_csr_build(_t(src), _t(dst), None, n, flags)
    starts = rng.integers(0, n, 1500).astype(np.int32)
    h_walks = oracle.random_walk(off, nb, starts, walk_len, seed=21)
    walks = gs.gs_random_walk(g, None, _t(starts), walk_len, 21)
    np.testing.assert_array_equal(walks.cpu().numpy(), h_walks)
    assert (h_walks[:, 1] < 0).any() and (h_walks[:, -1] >= 0).any()
    hc, ho = oracle.make_pairs(h_walks, window)
    total = hc.size
    offsets = gs.gs_pair_offsets(walks, window)
    per_walk = np.array([oracle.make_pairs(h_walks[i:i + 1], window)[0].size for i in range(len(starts))])
    np.testing.assert_array_equal(offsets.cpu().numpy(), np.concatenate([[0], np.cumsum(per_walk)]))
    nw = inputs.noise_weights(torch.as_tensor(off)).numpy()
    seg = np.array([0, n], dtype=np.int32)
    noise_h = oracle.alias_build(seg, nw)
    noise_d = gs.gs_alias_build(_t(seg), _t(nw), pack=True)
    f_in, f_out = inputs.random_tables(n, dim, seed=window, scale=0.2)
    if dtype == "bf16":
        d_in, d_out = f_in.to(torch.bfloat16).to(DEV), f_out.to(torch.bfloat16).to(DEV)
        h_in, h_out = _bf16_bits(d_in).copy(), _bf16_bits(d_out).copy()
        code = oracle.BF16
    else:
        d_in, d_out = f_in.to(DEV), f_out.to(DEV)
        h_in, h_out = f_in.numpy().copy(), f_out.numpy().copy()
        code = oracle.F32
    cuts = sorted({0, 1, 7, total // 3 + 1, total // 3 + 2, 2 * total // 3 + 5, total})
    base = (1 << 33) + 5
    for lo, hi in zip(cuts[:-1], cuts[1:]):
        m = hi - lo
        neg = oracle.sample_negatives(noise_h, n, m, k, seed=77, pair_index_base=base + lo)
        if k == 0:
            neg = np.zeros((m, 0), dtype=np.int32)
        want = oracle.sgns_step(h_in, h_out, hc[lo:hi], ho[lo:hi], neg, 0.02, dtype=code)
        loss = gs.gs_sgns_step_from_walks(d_in, d_out, walks, window, offsets, lo, m, noise_d, k, 77,
                                          0.02, pair_index_base=base + lo)
        torch.cuda.synchronize()
        assert abs(float(loss.item()) - want) <= LOSS_RTOL * abs(want)
        if dtype == "bf16":
            for d_t, h_t in ((d_in, h_in), (d_out, h_out)):
                # small batches touch few elements: one that rounds the other way weighs more
                assert_half_close(_bf16_bits(d_t), h_t, "bf16", flip_fraction=1e-3)
                d_t.copy_(torch.from_numpy(h_t.view(np.int16)).view(torch.bfloat16))
        else:
            assert np.abs(d_in.cpu().numpy() - h_in).max() <= EMB_ATOL
            assert np.abs(d_out.cpu().numpy() - h_out).max() <= EMB_ATOL
            d_in.copy_(torch.from_numpy(h_in))
            d_out.copy_(torch.from_numpy(h_out))
    # a slice that reaches past the last pair is reported through the loss
    loss = gs.gs_sgns_step_from_walks(d_in, d_out, walks, window, offsets, total - 3, 10, noise_d, k, 77, 0.02)
    assert np.isnan(float(loss.item()))
    # offsets that are not the numbering of these walks (every count doubled): reported the same
    # way, and no position outside a walk's live prefix is read
    other = offsets * 2
    loss = gs.gs_sgns_step_from_walks(d_in, d_out, walks, window, other, 0, min(total, 4096), noise_d, k, 77, 0.02)
    torch.cuda.synchronize()
    assert np.isnan(float(loss.item()))
