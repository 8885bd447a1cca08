"""The way that a batch takes with all the room it asks for, timed against the one that a little less room leaves it (sorted records,
or counters): batches of walks and negatives on few nodes, whose frequent ids have tens of thousands of terms.  The step of one table against that
of two."""
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def _batch(n, b, k, window):
    from paper_2407_15452_amd import binding as gs, inputs
    flags = gs.GS_SYMMETRIZE | gs.GS_DROP_SELF_LOOPS | gs.GS_DEDUPE
    wl = inputs.Workload("speed", "rmat", n, 10 * n, False, 32, 1, 1, 1, 1, 4, "f32", 0.025, False, 1, graph_seed=3)
    src, dst, _ = inputs.edge_list(wl, DEV)
    g = gs.gs_csr_build(src, dst, None, n, flags)
    noise = gs.gs_alias_build(torch.tensor([0, n], dtype=torch.int64, device=DEV), inputs.noise_weights(g.offsets))
    walks = gs.gs_random_walk(g, None, inputs.walk_starts(n, 0, 4 * b // window // 20 + 16, DEV), 40, 5)
    c, o, pairs = gs.gs_make_pairs(walks, window)
    assert pairs >= b
    return c[:b], o[:b], gs.gs_sample_negatives(noise, n, b, k, 7)


# buckets of rows that are split among workgroups; slices of long rows, of which many start nothing
@pytest.mark.parametrize("n,b,k,window,dim", [(5_000, 666_666, 5, 10, 52), (8_000, 600_000, 5, 10, 20),
                                              (5_000, 666_666, 10, 10, 20), (5_000, 600_000, 1, 10, 104)])
def test_no_slower_than_with_less_room(n, b, k, window, dim):
    from paper_2407_15452_amd import binding as gs, inputs
    batch = _batch(n, b, k, window)
    tabs = [t.to(DEV) for t in inputs.random_tables(n, dim, 3, 0.3)]
    size = gs.gs_sgns_step_workspace_bytes(b, n, k, dim, gs.GS_F32)
    ws = torch.empty(size, dtype=torch.uint8, device=DEV)
    loss = torch.zeros(1, dtype=torch.float64, device=DEV)
    times = {size: [], size - 256: []}
    for turn in range(12):
        for room, taken in times.items():
            first, last = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            first.record()
            for _ in range(5):
                gs.gs_sgns_step(*tabs, *batch, 1e-6, loss_out=loss, ws=ws[:room])
            last.record()
            torch.cuda.synchronize()
            if turn >= 2:
                taken.append(first.elapsed_time(last) / 5)
    own, less = (sorted(t)[len(t) // 2] for t in times.values())
    print("all room %.4f ms, less %.4f" % (own, less))
    assert own <= 1.08 * less, (own, less)       # (0.95 to 1.02, and 1.10 and more with what is named above; medians differ by about 0.01)


def test_one_table_keeps_its_rows_as_they_are_read():
    """The forward kernel of one table writes down every row of a centre that it reads; reading it twice for that costs 8 % of a step of 16-bit
    rows that do not fill the lanes (323 us against 298; the step of two tables takes 279)."""
    from paper_2407_15452_amd import binding as gs
    n, b, k, dim = 1_200_000, 68_603, 3, 392
    gen = torch.Generator(device=DEV).manual_seed(1)
    src = (torch.rand(b, generator=gen, device=DEV) * n).to(torch.int32).sort().values
    dst, neg = ((torch.rand(shape, generator=gen, device=DEV) * n).to(torch.int32) for shape in ((b,), (b, k)))
    tabs = [torch.rand((n, dim), generator=gen, device=DEV).sub_(0.5).to(torch.bfloat16) for _ in range(2)]
    loss = torch.zeros(1, dtype=torch.float64, device=DEV)
    ws = torch.empty(gs.gs_line1_step_workspace_bytes(b, n, k, dim, gs.GS_BF16), dtype=torch.uint8, device=DEV)
    calls = [lambda: gs.gs_line1_step(tabs[0], src, dst, neg, 1e-6, loss_out=loss, ws=ws),
             lambda: gs.gs_sgns_step(*tabs, src, dst, neg, 1e-6, loss_out=loss, ws=ws)]
    times = ([], [])
    for turn in range(12):
        for call, taken in zip(calls, times):
            first, last = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            first.record()
            for _ in range(5):
                call()
            last.record()
            torch.cuda.synchronize()
            if turn >= 2:
                taken.append(first.elapsed_time(last) / 5)
    one, two = (sorted(t)[len(t) // 2] for t in times)
    print("one table %.4f ms, two %.4f" % (one, two))
    assert one <= 1.115 * two, (one, two)
