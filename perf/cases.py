"""The work that programs built on this library have it do, as cases that can be timed.

Each case is one call, or the few calls that belong together, through the public entry points
of ``paper_2407_15452_amd.binding``: the training iteration in its variants, the walks, the pairs
and negatives made from them, the LINE batch, the storage operations and the building of the
graph and its alias tables.  Inputs are synthetic: R-MAT graphs from
``paper_2407_15452_amd.inputs`` (the recipe of the benchmark's workloads), walks on them, pairs
of those walks and negatives from the degree**0.75 table, so that ids repeat as they do in
training; the tables hold mid-training values.
"""
from __future__ import annotations

import math

import torch

from paper_2407_15452_amd import binding as gs, inputs

DEV = "cuda:0"
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
FLAGS = gs.GS_SYMMETRIZE | gs.GS_DROP_SELF_LOOPS | gs.GS_DEDUPE


def _batch(name, pairs, nodes, edges, dim, dtype, k, **more):
    case = {"op": "step", "call": "step", "pairs": pairs, "nodes": nodes, "edges": edges, "dim": dim, "dtype": dtype,
            "k": k, "walk_len": 40, "window": 5, "node2vec": False}
    case.update(more)
    if name:
        case["name"] = name
    return case


def _walk(name, kind, walks, walk_len, nodes, edges, offset_bits=32):
    case = {"op": "walk", "kind": kind, "walks": walks, "walk_len": walk_len, "nodes": nodes, "edges": edges,
            "offset_bits": offset_bits}
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # the small batches of the paper (512 to 2048 sources) on a graph much larger than the
        # batch: latency and the number of launches count
        _batch("step-small", 2048, 1_000_000, 10_000_000, 128, "f32", 5),
        # the benchmark's smallest workload: DeepWalk on 10,000 nodes, 65,536 pairs, narrow rows
        _batch("step-64k", 65_536, 10_000, 100_000, 64, "f32", 5, walk_len=20),
        # the benchmark's default workload: node2vec walks on 4 million nodes, 2 million pairs
        _batch("step-2m", 2_000_000, 4_000_000, 64_000_000, 128, "f32", 5, walk_len=80, window=10, node2vec=True),
        # the recommender setting: 16-bit tables, wide rows, ten negatives
        _batch("step-bf16", 1_000_000, 4_000_000, 20_000_000, 256, "bf16", 10),
        # the paper's optimizers: SGD with momentum and Adam inside the storage (dense passes over
        # every table around the sparse update)
        _batch("momentum", 262_144, 1_000_000, 10_000_000, 128, "f32", 5, call="momentum"),
        _batch("adam", 262_144, 1_000_000, 10_000_000, 128, "f32", 5, call="adam"),
        # a LINE batch (edges sampled, sorted by source, negatives, iteration), ragged sizes, fp16 tables
        {"op": "line", "name": "line-f16-ragged", "order": 2, "pairs": 300_007, "nodes": 777_777, "edges": 5_000_000,
         "dim": 200, "dtype": "f16", "k": 7, "weighted": False},
        # node2vec walks, a chunk that feeds some twenty batches of the default workload
        _walk("walk-node2vec", "node2vec", 47_000, 80, 4_000_000, 64_000_000),
        # weighted first-order walks from every node
        _walk("walk-weighted", "weighted", 1_000_000, 40, 1_000_000, 10_000_000),
        # skip-gram pairs of a chunk of walks and the negatives of one batch
        {"op": "pairs", "name": "pairs-negatives", "walks": 30_000, "walk_len": 80, "window": 10, "nodes": 1_000_000,
         "edges": 10_000_000, "pairs": 2_000_000, "k": 5},
        # topology and tables of a program's start: CSR, per-row alias tables, noise table
        {"op": "build", "name": "build", "nodes": 1_000_000, "edges": 10_000_000, "weighted": True, "offset_bits": 32},
        # the storage operations of one batch: merged ids, get of the rows, put of their gradients
        {"op": "storage", "name": "storage", "ids": 2_000_000, "nodes": 4_000_000, "edges": 20_000_000, "dim": 128,
         "dtype": "f32"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["step"] * 6 + ["walk"] * 3 + ["pairs", "line", "line", "storage", "build"])
    nodes = _log(rng, 5_000, 2_000_000)
    edges = int(nodes * rng.uniform(4, 14))
    dtype = rng.choice(["f32", "f32", "bf16", "f16"])
    granule = 4 if dtype == "f32" else 8
    dim = max(granule, int(round(_log(rng, 16, 400) / granule)) * granule)
    k = rng.choice([1, 2, 3, 5, 5, 5, 7, 10, 15])
    most = max(256, int(min(1_000_000, 1.2e9 / ((k + 1) * dim))))
    pairs = _log(rng, 256, most)
    walk_len = rng.choice([10, 20, 33, 40, 80])
    window = rng.choice([2, 3, 5, 10])
    if op == "step":
        call = rng.choice(["step", "step", "step", "from_walks", "fused", "static", "momentum", "adam"])
        if call == "static":
            pairs, dim = min(pairs, 4096), min(dim, 256)
        if call == "adam":
            dtype = "f32"
        return _batch(None, pairs, nodes, edges, dim, dtype, k, call=call, walk_len=walk_len, window=window,
                      node2vec=rng.random() < 0.3)
    if op == "walk":
        return _walk(None, rng.choice(["uniform", "weighted", "node2vec", "node2vec"]), _log(rng, 200, 1_000_000),
                     walk_len, nodes, edges, rng.choice([32, 32, 64]))
    if op == "pairs":
        return {"op": "pairs", "walks": _log(rng, 200, 30_000), "walk_len": walk_len, "window": window, "nodes": nodes,
                "edges": edges, "pairs": _log(rng, 256, 2_000_000), "k": k}
    if op == "line":
        return {"op": "line", "order": rng.choice([1, 2]), "pairs": pairs, "nodes": nodes, "edges": edges, "dim": dim,
                "dtype": dtype, "k": k, "weighted": rng.random() < 0.5}
    if op == "storage":
        return {"op": "storage", "ids": _log(rng, 500, max(1000, int(min(2_000_000, 2e8 / dim)))), "nodes": nodes,
                "edges": edges, "dim": dim, "dtype": dtype}
    return {"op": "build", "nodes": min(nodes, 1_000_000), "edges": min(edges, 10_000_000),
            "weighted": rng.random() < 0.5, "offset_bits": rng.choice([32, 64])}


# ---- inputs ---------------------------------------------------------------------------------
def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _edges(case, seed):
    wl = inputs.Workload("case", "rmat", case["nodes"], case["edges"], False, 32, 1, 1, 1, 1, 4, "f32", 0.025, False, 1,
                         graph_seed=seed * 2654435761 + 0x67530100)
    src, dst, _ = inputs.edge_list(wl, DEV)
    return src, dst


def _weights(n, gen):
    # lognormal(0, 1), as the interactions of the benchmark's bipartite workload
    return torch.exp(torch.randn(n, generator=gen, device=DEV))


def _graph(case, seed, gen, weighted=False):
    src, dst = _edges(case, seed)
    w = _weights(src.numel(), gen) if weighted else None
    return gs.gs_csr_build(src, dst, w, case["nodes"], FLAGS, case.get("offset_bits", 32))


def _segment(n):
    return torch.tensor([0, n], dtype=torch.int64, device=DEV)


def _noise(g):
    return gs.gs_alias_build(_segment(g.num_nodes), inputs.noise_weights(g.offsets))


def _table(case, gen):
    t = torch.rand((case["nodes"], case["dim"]), generator=gen, device=DEV)
    return t.sub_(0.5).to(DTYPES[case["dtype"]])


def _walks_for(g, case, seed, pairs):
    """Walks (consecutive starts) that hold at least `pairs` pairs, and their pairs."""
    per = inputs.pairs_per_full_walk(case["walk_len"], case["window"])
    count = int(pairs / per * 2) + 16
    while True:
        starts = inputs.walk_starts(g.num_nodes, (seed * 7919) % g.num_nodes, count, DEV)
        if case["node2vec"]:
            walks = gs.gs_node2vec_walk(g, None, starts, case["walk_len"], 0.5, 2.0, seed)
        else:
            walks = gs.gs_random_walk(g, None, starts, case["walk_len"], seed)
        centers, contexts, n = gs.gs_make_pairs(walks, case["window"])
        if n >= pairs:
            return walks, centers, contexts, n
        count *= 2


def _rate(pairs):
    return 0.025 * min(1.0, inputs.LR_REFERENCE_PAIRS / pairs)


BETA1, BETA2, EPS, ADAM_T, MU = 0.9, 0.999, 1e-8, 10, 0.9
ADAM_LR = 1e-3


def _dtype_code(case):
    return {"f32": gs.GS_F32, "bf16": gs.GS_BF16, "f16": gs.GS_F16}[case["dtype"]]


def prepare(case, seed):
    gen = _generator(seed)
    op = case["op"]
    s = {"case": case, "seed": seed}
    if op == "build":
        # one graph, its vertices renamed and its edge list shuffled by the seed (the number of
        # distinct edges, and with it the shape of what comes out, is then the same for every seed)
        src, dst = _edges(case, 1)
        rename = torch.randperm(case["nodes"], generator=gen, device=DEV)
        order = torch.randperm(src.numel(), generator=gen, device=DEV)
        src, dst = rename[src[order].long()].to(torch.int32), rename[dst[order].long()].to(torch.int32)
        w = _weights(src.numel(), gen) if case["weighted"] else None
        g = gs.gs_csr_build(src, dst, w, case["nodes"], FLAGS, case["offset_bits"])
        s.update(src=src, dst=dst, w=w, noise_w=inputs.noise_weights(g.offsets), seg=_segment(case["nodes"]))
        return s
    weighted = case.get("kind") == "weighted" or (op == "line" and case["weighted"])
    g = _graph(case, seed, gen, weighted)
    if op == "walk":
        s.update(g=g, rows=gs.gs_alias_build(g.offsets, g.weights) if weighted else None,
                 starts=inputs.walk_starts(case["nodes"], (seed * 7919) % case["nodes"], case["walks"], DEV))
        return s
    noise = _noise(g)
    if op == "pairs":
        starts = inputs.walk_starts(case["nodes"], (seed * 7919) % case["nodes"], case["walks"], DEV)
        room = max(1, gs.pair_capacity(case["walks"], case["walk_len"], case["window"]))
        s.update(walks=gs.gs_random_walk(g, None, starts, case["walk_len"], seed), noise=noise,
                 centers=torch.zeros(room, dtype=torch.int32, device=DEV),
                 contexts=torch.zeros(room, dtype=torch.int32, device=DEV),
                 count=torch.zeros(1, dtype=torch.int64, device=DEV))
        return s
    if op == "storage":
        ids = gs.gs_sample_negatives(noise, case["nodes"], case["ids"], 1, seed).view(-1)
        n = case["ids"]
        s.update(ids=ids, table=_table(case, gen), out=torch.zeros((n, case["dim"]), device=DEV),
                 grads=torch.randn((n, case["dim"]), generator=gen, device=DEV).mul_(0.1))
        return s
    pairs, nodes, k, dim = case["pairs"], case["nodes"], case["k"], case["dim"]
    s.update(noise=noise, w_in=_table(case, gen), w_out=_table(case, gen),
             loss=torch.zeros(1, dtype=torch.float64, device=DEV),
             negs=torch.empty((pairs, k), dtype=torch.int32, device=DEV))
    code = _dtype_code(case)
    if op == "line":
        s.update(g=g, edges=gs.gs_alias_build(_segment(g.num_entries), g.weights) if weighted else None)
        if case["order"] == 1:
            need = gs.gs_line1_step_workspace_bytes(pairs, nodes, k, dim, code)
        else:
            need = gs.gs_sgns_step_workspace_bytes(pairs, nodes, k, dim, code)
        s["ws"] = torch.empty(max(need, 256), dtype=torch.uint8, device=DEV)
        return s
    walks, centers, contexts, n = _walks_for(g, case, seed, pairs)
    lo = (seed * 104729) % (n - pairs + 1)
    s.update(lo=lo, centers=centers[lo:lo + pairs].clone(), contexts=contexts[lo:lo + pairs].clone())
    call = case["call"]
    if call == "from_walks":
        s.update(walks=walks, pair_offsets=gs.gs_pair_offsets(walks, case["window"]))
        need = gs.gs_sgns_step_from_walks_workspace_bytes(pairs, nodes, k, dim, code)
    elif call == "fused":
        need = gs.gs_sgns_step_fused_workspace_bytes(pairs, nodes, k, dim, code)
    else:
        need = gs.gs_sgns_step_workspace_bytes(pairs, nodes, k, dim, code)
    s["ws"] = torch.empty(max(need, 256), dtype=torch.uint8, device=DEV)
    if call in ("momentum", "adam"):
        for name in ("m_in", "m_out"):
            s[name] = torch.randn((nodes, dim), generator=gen, device=DEV).mul_(1e-2).to(DTYPES[case["dtype"]])
    if call == "adam":
        for name in ("v_in", "v_out"):
            s[name] = torch.rand((nodes, dim), generator=gen, device=DEV).mul_(1e-2).add_(1e-3)
    return s


def run(s):
    case, seed = s["case"], s["seed"]
    op = case["op"]
    if op == "build":
        g = gs.gs_csr_build(s["src"], s["dst"], s["w"], case["nodes"], FLAGS, case["offset_bits"])
        noise = gs.gs_alias_build(s["seg"], s["noise_w"])
        out = {"offsets": g.offsets, "nbrs": g.nbrs, "noise_prob": noise.prob, "noise_alias": noise.alias,
               "noise_packed": noise.packed}
        if case["weighted"]:
            rows = gs.gs_alias_build(g.offsets, g.weights)
            out.update(weights=g.weights, prob=rows.prob, alias=rows.alias, packed=rows.packed)
        return out
    if op == "walk":
        if case["kind"] == "node2vec":
            return gs.gs_node2vec_walk(s["g"], None, s["starts"], case["walk_len"], 0.5, 2.0, seed)
        return gs.gs_random_walk(s["g"], s["rows"], s["starts"], case["walk_len"], seed)
    if op == "pairs":
        centers, contexts, n = gs.gs_make_pairs(s["walks"], case["window"], s["centers"], s["contexts"], s["count"],
                                                sync=False)
        return {"centers": centers, "contexts": contexts, "n": n,
                "negs": gs.gs_sample_negatives(s["noise"], case["nodes"], case["pairs"], case["k"], seed)}
    if op == "storage":
        unique, count, inverse = gs.gs_unique_ids(s["ids"], case["nodes"])
        rows = gs.gs_get_rows(s["table"], unique, count, out=s["out"])   # row i is the row of the i-th merged id
        gs.gs_put_rows(s["table"], unique, s["grads"], -0.025, count)
        return {"count": count, "inverse": inverse, "rows": rows, "table": s["table"]}
    pairs, nodes, k = case["pairs"], case["nodes"], case["k"]
    lr = _rate(pairs)
    if op == "line":
        src, dst = gs.gs_sample_edges(s["g"], s["edges"], pairs, seed)
        src, dst = gs.gs_sort_pairs(src, dst, nodes)
        negs = gs.gs_sample_negatives(s["noise"], nodes, pairs, k, seed + 1, out=s["negs"])
        if case["order"] == 1:
            loss = gs.gs_line1_step(s["w_in"], src, dst, negs, lr, loss_out=s["loss"], ws=s["ws"])
            return {"w": s["w_in"], "loss": loss}
        loss = gs.gs_sgns_step(s["w_in"], s["w_out"], src, dst, negs, lr, loss_out=s["loss"], ws=s["ws"])
        return {"w_in": s["w_in"], "w_out": s["w_out"], "loss": loss}
    call = case["call"]
    out = {"w_in": s["w_in"], "w_out": s["w_out"]}
    if call == "from_walks":
        out["loss"] = gs.gs_sgns_step_from_walks(s["w_in"], s["w_out"], s["walks"], case["window"], s["pair_offsets"],
                                                 s["lo"], pairs, s["noise"], k, seed, lr, loss_out=s["loss"],
                                                 ws=s["ws"])
        return out
    if call == "fused":
        out["loss"] = gs.gs_sgns_step_fused(s["w_in"], s["w_out"], s["centers"], s["contexts"], s["noise"], k, seed,
                                            lr, loss_out=s["loss"], ws=s["ws"])
        return out
    negs = gs.gs_sample_negatives(s["noise"], nodes, pairs, k, seed, out=s["negs"])
    if call == "static":
        out["loss"] = gs.gs_sgns_step_static(s["w_in"], s["w_out"], s["centers"], s["contexts"], negs, lr,
                                             loss_out=s["loss"])
    elif call == "momentum":
        out["loss"] = gs.gs_sgns_momentum_step(s["w_in"], s["w_out"], s["m_in"], s["m_out"], s["centers"],
                                               s["contexts"], negs, lr, MU, loss_out=s["loss"], ws=s["ws"])
        out.update(m_in=s["m_in"], m_out=s["m_out"])
    elif call == "adam":
        out["loss"] = gs.gs_sgns_adam_step(s["w_in"], s["w_out"], s["m_in"], s["m_out"], s["v_in"], s["v_out"],
                                           s["centers"], s["contexts"], negs, ADAM_LR, BETA1, BETA2, EPS, ADAM_T,
                                           loss_out=s["loss"], ws=s["ws"])
        out.update(m_in=s["m_in"], m_out=s["m_out"], v_in=s["v_in"], v_out=s["v_out"])
    else:
        out["loss"] = gs.gs_sgns_step(s["w_in"], s["w_out"], s["centers"], s["contexts"], negs, lr,
                                      loss_out=s["loss"], ws=s["ws"])
    return out


# ---- what a pass cannot do without ----------------------------------------------------------
LIVE = 0.65     # share of the nodes of these graphs that have edges; of walk positions that are visited


def _distinct(draws, nodes):
    """Distinct rows among `draws` ids of a graph's live nodes (equally likely ids)."""
    live = max(1.0, LIVE * nodes)
    return live * -math.expm1(-draws / live)


def work(case):
    op = case["op"]
    n = case["nodes"]
    if op == "walk":
        steps = LIVE * case["walks"] * (case["walk_len"] - 1)
        per = case["offset_bits"] // 8 * 2 + 4 + (8 if case["kind"] == "weighted" else 0)
        return {"bytes": 4 * case["walks"] * (case["walk_len"] + 1) + steps * per, "flops": 0}
    if op == "pairs":
        made = LIVE * case["walks"] * inputs.pairs_per_full_walk(case["walk_len"], case["window"])
        return {"bytes": 4 * case["walks"] * case["walk_len"] + 8 * made + 12 * case["pairs"] * case["k"], "flops": 0}
    if op == "build":
        e = 2 * case["edges"]
        per = 8 + 4 + ((4 + 4 + 8 + 8) if case["weighted"] else 0)
        return {"bytes": e * per + n * (case["offset_bits"] // 8 + 4 + 8 + 8), "flops": 0}
    rb = case["dim"] * (4 if case["dtype"] == "f32" else 2)
    if op == "storage":
        u = _distinct(case["ids"], n)
        return {"bytes": 8 * case["ids"] + u * (2 * rb + 2 * 4 * case["dim"]), "flops": 2 * u * case["dim"]}
    pairs, k = case["pairs"], case["k"]
    flops = 6.0 * pairs * (k + 1) * case["dim"]
    index = 4.0 * pairs * (2 + 2 * k)
    contexts = _distinct(pairs * (k + 1), n)
    if op == "line":
        centers = _distinct(pairs, n)
        rows = _distinct(pairs * (k + 2), n) if case["order"] == 1 else contexts + centers
        return {"bytes": index + 2 * rows * rb, "flops": flops}
    if case["call"] == "momentum":
        return {"bytes": index + 8.0 * n * rb, "flops": flops}
    if case["call"] == "adam":
        return {"bytes": index + 12.0 * n * rb, "flops": flops}
    centers = _distinct(pairs / (2 * case["window"]), n)
    return {"bytes": index + 2 * (contexts + centers) * rb, "flops": flops}


def tolerance(case):
    # walks, pairs, negatives, graphs, alias tables and the storage operations are defined bit for
    # bit; a training iteration differs by the order of a logit's fp32 sum
    if case["op"] not in ("step", "line"):
        return "exact"
    if case["op"] == "step" and case["call"] == "adam":     # (1 - beta2 in fp32, and a quotient and a root per element)
        return {"rel": 1.5e-5, "max": 1e-3}
    if case["dtype"] == "f32":
        return {"rel": 5e-7, "max": 1e-4}
    # 16-bit tables: one rounding per written element, so a result on a rounding boundary may fall
    # the other way (one 16-bit step; about 2e-5 of the elements in bf16, 2e-4 in fp16)
    return {"rel": 2e-4, "max": 1.6e-2}


# ---- the same in 64 bits, in plain torch ------------------------------------------------------
def _philox(seed, index, c2, c3):
    """Words 0..2 of the Philox4x32-10 block with key `seed` and counter (index, c2, c3), as int64."""
    mask = 0xFFFFFFFF
    c = [index & mask, (index >> 32) & mask, c2 + 0 * index, c3 + 0 * index]
    k0, k1 = seed & mask, (seed >> 32) & mask
    for _ in range(10):
        a, b = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57     # (wraps as unsigned 64-bit products do)
        c = [((b >> 32) & mask) ^ c[1] ^ k0, b & mask, ((a >> 32) & mask) ^ c[3] ^ k1, a & mask]
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    return c[0], c[1], c[2]


def _alias_draw(table, n, words):
    """slot = high half of (word0, word1) * n; the slot's alias unless word2 falls below its prob."""
    x0, x1, x2 = words
    at = (x0 * n + ((x1 * n) >> 32)) >> 32
    if table is None:
        return at
    keep = (x2 >> 8).float() * 2.0 ** -24 < table.prob[at]
    return torch.where(keep, at, table.alias[at].long())


def _negatives(noise, nodes, pairs, k, seed):
    i = torch.arange(pairs, device=DEV)
    return torch.stack([_alias_draw(noise, nodes, _philox(seed, i, j, 0x80000000)) for j in range(k)], 1)


def _gradients(w_in, w_out, centers, contexts, negs):
    """Loss and gradients (summed over the batch) of both tables, in 64 bits."""
    d_in = torch.zeros(w_in.shape, dtype=torch.float64, device=DEV)
    d_out = torch.zeros(w_out.shape, dtype=torch.float64, device=DEV)
    loss = torch.zeros(1, dtype=torch.float64, device=DEV)
    k1, dim = negs.shape[1] + 1, w_in.shape[1]
    step = max(1, int(6e7 // (k1 * dim)))
    for lo in range(0, centers.numel(), step):
        c = centers[lo:lo + step].long()
        rows = torch.cat([contexts[lo:lo + step].long()[:, None], negs[lo:lo + step].long()], 1)
        u, v = w_in[c].double(), w_out[rows].double()
        x = (v * u[:, None, :]).sum(-1)
        sign = torch.ones_like(x)
        sign[:, 0] = -1.0
        loss += torch.nn.functional.softplus(sign * x).sum()
        g = torch.sigmoid(x)
        g[:, 0] -= 1.0
        d_in.index_add_(0, c, (g[:, :, None] * v).sum(1))
        d_out.index_add_(0, rows.reshape(-1), (g[:, :, None] * u[:, None, :]).reshape(-1, dim))
    return loss, d_in, d_out


def exact(case, seed):
    op = case["op"]
    if op in ("walk", "pairs", "build"):
        return None         # whole numbers and tables that are defined bit for bit
    s = prepare(case, seed)
    if op == "storage":
        unique, inverse = torch.unique(s["ids"].long(), return_inverse=True)
        rows = torch.zeros((case["ids"], case["dim"]), dtype=torch.float64, device=DEV)
        rows[:unique.numel()] = s["table"][unique].double()
        table = s["table"].double()
        table[unique] += -0.025 * s["grads"][:unique.numel()].double()
        return {"count": None, "inverse": None, "rows": rows, "table": table}
    pairs, nodes, k = case["pairs"], case["nodes"], case["k"]
    lr = _rate(pairs)
    if op == "line":
        g = s["g"]
        entry = _alias_draw(s["edges"], g.num_entries, _philox(seed, torch.arange(pairs, device=DEV), 0, 0x40000000))
        src, dst = torch.searchsorted(g.offsets, entry.to(g.offsets.dtype), right=True) - 1, g.nbrs[entry]
        order = torch.argsort(src, stable=True)
        src, dst = src[order], dst[order]
        negs = _negatives(s["noise"], nodes, pairs, k, seed + 1)
        w_out = s["w_in"] if case["order"] == 1 else s["w_out"]
        loss, d_in, d_out = _gradients(s["w_in"], w_out, src, dst, negs)
        if case["order"] == 1:
            return {"w": s["w_in"].double() - lr * (d_in + d_out), "loss": loss}
        return {"w_in": s["w_in"].double() - lr * d_in, "w_out": w_out.double() - lr * d_out, "loss": loss}
    negs = _negatives(s["noise"], nodes, pairs, k, seed)
    loss, d_in, d_out = _gradients(s["w_in"], s["w_out"], s["centers"], s["contexts"], negs)
    if case["call"] == "momentum":
        m_in, m_out = MU * s["m_in"].double() + d_in, MU * s["m_out"].double() + d_out
        return {"w_in": s["w_in"].double() - lr * m_in, "w_out": s["w_out"].double() - lr * m_out, "loss": loss,
                "m_in": m_in, "m_out": m_out}
    if case["call"] == "adam":
        out = {"loss": loss}
        for side, d in (("in", d_in), ("out", d_out)):
            m = BETA1 * s["m_" + side].double() + (1 - BETA1) * d
            v = BETA2 * s["v_" + side].double() + (1 - BETA2) * d * d
            move = ADAM_LR / (1 - BETA1 ** ADAM_T) * m / (v.sqrt() / math.sqrt(1 - BETA2 ** ADAM_T) + EPS)
            out.update({"w_" + side: s["w_" + side].double() - move, "m_" + side: m, "v_" + side: v})
        return out
    return {"w_in": s["w_in"].double() - lr * d_in, "w_out": s["w_out"].double() - lr * d_out, "loss": loss}
