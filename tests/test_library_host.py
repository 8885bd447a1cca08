"""CPU-side checks of the HIP library: it loads, exports every symbol declared
in include/gs.h, and its host-only functions (workspace sizing) behave.  No
kernel is launched here."""
import ctypes as C
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    from paper_2407_15452_amd import binding, build
    if not os.path.exists(binding.LIB_PATH):
        build.build_lib()
    return binding.lib()


def test_header_symbols_are_exported(lib):
    from paper_2407_15452_amd import binding
    header = open(os.path.join(ROOT, "include", "gs.h")).read()
    declared = set(re.findall(r"\b(gs_[a-z0-9_]+)\s*\(", header))
    assert declared == set(binding.EXPORTS)
    for name in declared:
        assert getattr(lib, name) is not None


def test_workspace_queries(lib):
    assert lib.gs_sgns_step_workspace_bytes(C.c_int64(0), C.c_int64(10), C.c_int32(5), C.c_int32(128), C.c_int32(0)) > 0
    small = lib.gs_sgns_step_workspace_bytes(C.c_int64(1000), C.c_int64(10), C.c_int32(5), C.c_int32(128), C.c_int32(0))
    big = lib.gs_sgns_step_workspace_bytes(C.c_int64(2000), C.c_int64(10), C.c_int32(5), C.c_int32(128), C.c_int32(0))
    assert 0 < small < big and small % 256 == 0
    assert lib.gs_csr_build_workspace_bytes(C.c_int64(1000), C.c_int64(10), C.c_uint32(1)) > \
        lib.gs_csr_build_workspace_bytes(C.c_int64(1000), C.c_int64(10), C.c_uint32(0))
    assert lib.gs_make_pairs_workspace_bytes(C.c_int64(10)) >= 256
    assert lib.gs_alias_build_workspace_bytes(C.c_int64(3), C.c_int64(100)) >= 16 * 100
    assert lib.gs_last_hip_error() == 0


def test_missing_library_is_an_error(monkeypatch):
    from paper_2407_15452_amd import binding
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "LIB_PATH", "/nonexistent/libgs.so")
    with pytest.raises(RuntimeError):
        binding.lib()


def test_bench_refuses_more_than_one_gpu():
    import subprocess
    import sys
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True)
    assert r.returncode != 0 and "one GPU" in r.stderr


def test_inputs_are_deterministic():
    import torch
    from paper_2407_15452_amd import inputs
    wl = inputs.WORKLOADS[0]
    a = inputs.edge_list(wl)
    b = inputs.edge_list(wl)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]) and a[0].numel() == wl.num_edges
    assert inputs.pairs_per_full_walk(20, 5) == 170 and inputs.pairs_per_full_walk(80, 10) == 1490
    w_in, w_out = inputs.init_tables(100, 64, 5)
    assert float(w_in.abs().max()) <= 0.5 / 64 and float(w_out.abs().max()) == 0


def test_argument_checks_that_need_no_gpu(lib):
    """Rejected on the host before anything is enqueued (no device pointer is touched)."""
    fake = C.c_void_p(256)                       # non-null, aligned; never dereferenced
    # one alias segment longer than a 32-bit position
    rc = lib.gs_alias_build(fake, C.c_int32(64), C.c_int64(1), C.c_int64(1 << 31), fake, fake, fake,
                            fake, C.c_size_t(1 << 62), None)
    assert rc == -3
    # 32-bit offsets cannot hold the symmetrised capacity
    rc = lib.gs_csr_build(fake, fake, None, C.c_int64((1 << 30) + 1), C.c_int64(10), C.c_uint32(1),
                          C.c_int32(32), fake, fake, None, fake, fake, C.c_size_t(1 << 62), None)
    assert rc == -3
    # dim not a multiple of the 16-byte piece; k beyond the limit; one table on both sides
    step = lambda w_in, w_out, dim, k: lib.gs_sgns_step(  # noqa: E731
        w_in, w_out, C.c_int64(10), C.c_int32(dim), C.c_int32(0), fake, fake, fake, C.c_int64(4),
        C.c_int32(k), C.c_float(0.1), fake, fake, C.c_size_t(1 << 62), None)
    other = C.c_void_p(512)
    assert step(fake, other, 6, 2) == -1
    assert step(fake, other, 8, 61) == -1
    assert step(fake, fake, 8, 2) == -1
    assert lib.gs_unique_ids_workspace_bytes(C.c_int64(1000), C.c_int64(100)) < \
        lib.gs_unique_ids_workspace_bytes(C.c_int64(1000), C.c_int64(10**9))
    assert lib.gs_sgns_step_fused_workspace_bytes(C.c_int64(1000), C.c_int64(10), C.c_int32(5), C.c_int32(128), C.c_int32(0)) > \
        lib.gs_sgns_step_workspace_bytes(C.c_int64(1000), C.c_int64(10), C.c_int32(5), C.c_int32(128), C.c_int32(0))


def test_static_step_rejects_oversized_batches_on_the_host(lib):
    """gs_sgns_step_static checks its limits before it asks for the scratch array's address."""
    fake, other = C.c_void_p(256), C.c_void_p(512)
    call = lambda pairs, k, dim: lib.gs_sgns_step_static(  # noqa: E731
        fake, other, C.c_int64(10), C.c_int32(dim), C.c_int32(0), fake, fake, fake, C.c_int64(pairs),
        C.c_int32(k), C.c_float(0.1), fake, None)
    assert call(4097, 5, 128) == -2
    assert call(4096, 16, 128) == -2            # 4096 * 17 terms > 65536
    assert call(1024, 5, 260) == -2


def test_workspace_sizes_beyond_two_gigabytes(lib):
    """Sizes are size_t all the way: a batch whose staged rows alone take more than 2^31 bytes."""
    for fn in (lib.gs_sgns_step_workspace_bytes, lib.gs_sgns_step_fused_workspace_bytes,
               lib.gs_sgns_step_from_walks_workspace_bytes, lib.gs_line1_step_workspace_bytes):
        for pairs, nodes, k, dim in ((2_000_000, 25_000_000, 10, 256), (4_000_000, 100_000_000, 5, 128),
                                     (3_000_000, 50_000, 1, 256)):
            staged = pairs * dim * 4
            size = fn(C.c_int64(pairs), C.c_int64(nodes), C.c_int32(k), C.c_int32(dim), C.c_int32(1))
            assert staged < size < 8 * staged


def test_workspace_for_many_records_serves_fewer(lib):
    """The sort takes larger tiles from 2^21 records on; what is asked for does not fall there."""
    queries = [lambda n: lib.gs_sort_pairs_workspace_bytes(C.c_int64(n)),
               lambda n: lib.gs_unique_ids_workspace_bytes(C.c_int64(n), C.c_int64(2_000_000_000)),
               lambda n: lib.gs_csr_build_workspace_bytes(C.c_int64(n), C.c_int64(1000), C.c_uint32(0)),
               lambda n: lib.gs_csr_build_workspace_bytes(C.c_int64(n // 2), C.c_int64(1000), C.c_uint32(1))]
    sizes = sorted({max(1, (1 << 21) + d) for d in (-200_000, -4096, -2049, -2, -1, 0, 1, 2048, 8193, 1 << 21, 3 << 21)}
                   | {1, 2047, 2048, 2049, 100_000, 1 << 28})
    for query in queries:
        got = [query(n) for n in sizes]
        assert got == sorted(got) and got[0] > 0


@pytest.mark.parametrize("pairs,nodes", [(1000, 1_000_000), (800_000, 3_000_000)])
def test_workspace_below_the_counters_plan_is_refused(lib, pairs, nodes):
    """Batches for which the counters' plan is the largest of those that the step may take (a small one, and one
    whose terms are sorted): with less, no call starts, whatever else would fit.  Nothing is enqueued."""
    k, dim, t = 5, 8, [C.c_void_p(256 * i) for i in range(1, 8)]
    n, b, dims = C.c_int64(nodes), C.c_int64(pairs), (C.c_int32(k), C.c_int32(dim), C.c_int32(0))
    lr, zero, null = C.c_float(0.1), C.c_uint64(0), None
    size = lambda fn: C.c_size_t(fn(b, n, *dims) - 256)  # noqa: E731
    table = (n, C.c_int32(dim), C.c_int32(0))
    assert lib.gs_sgns_step(t[0], t[1], *table, t[2], t[3], t[4], b, dims[0], lr, t[5], t[6],
                            size(lib.gs_sgns_step_workspace_bytes), null) == -2
    assert lib.gs_sgns_momentum_step(t[0], t[1], t[2], t[3], *table, t[2], t[3], t[4], b, dims[0], lr, lr, t[5], t[6],
                                     size(lib.gs_sgns_step_workspace_bytes), null) == -2
    assert lib.gs_sgns_step_fused(t[0], t[1], *table, t[2], t[3], b, null, zero, zero, dims[0], lr, t[5], t[6],
                                  size(lib.gs_sgns_step_fused_workspace_bytes), null) == -2
    assert lib.gs_sgns_step_from_walks(t[0], t[1], *table, t[2], C.c_int64(10), C.c_int32(5), C.c_int32(2), t[3],
                                       C.c_int64(0), b, null, zero, zero, dims[0], lr, t[5], t[6],
                                       size(lib.gs_sgns_step_from_walks_workspace_bytes), null) == -2
    assert lib.gs_line1_step(t[0], *table, t[2], t[3], t[4], b, dims[0], lr, t[5], t[6],
                             size(lib.gs_line1_step_workspace_bytes), null) == -2


@pytest.mark.parametrize("nodes", [1, 5, 300, 10_000, 18_431, 131_072, 131_073, 300_000, 4_000_000, 100_000_000])
def test_workspace_of_a_large_batch_serves_smaller_ones(lib, nodes):
    """What the training steps ask for never falls as the batch grows: over the ends of the two-launch step, of
    the table of the batch's keys and of the input keys, of short segments, and the start of the sorted records."""
    queries = (lib.gs_sgns_step_workspace_bytes, lib.gs_sgns_step_fused_workspace_bytes,
               lib.gs_sgns_step_from_walks_workspace_bytes, lib.gs_line1_step_workspace_bytes)
    for k, dim, dtype in ((0, 256, 0), (5, 256, 0), (5, 8, 1), (60, 512, 2)):
        ends = {1, 2, 1 << 18, 1 << 20, 49_152 // (k + 2), int((nodes << 17) ** 0.5) // (k + 2), nodes // 8 // (k + 2),
                (1 << 20) // (k + 1), (1 << 21) // (k + 1), (9 << 19) // (k + 1), (3 << 21) // (k + 1), 3_000_000}
        ends |= {1 << s for s in range(1, 22)}
        sizes = sorted({e + d for e in ends for d in (-1, 0, 1, 2) if e + d > 0 and (e + d) * (k + 1) < 1 << 31})
        for query in queries:
            got = [query(C.c_int64(b), C.c_int64(nodes), C.c_int32(k), C.c_int32(dim), C.c_int32(dtype)) for b in sizes]
            falls = [(b, x, y) for b, x, y in zip(sizes, got, got[1:]) if y < x]
            assert not falls, (k, dim, dtype, falls)
