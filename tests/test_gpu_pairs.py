"""Pair emission where its closed form changes: windows at, just below and just above half a walk
(with and without centres that have a full window on both sides), walks cut to every length, and
walk lengths at which fewer walks share a block."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("walk_len,window,walks", [(21, 10, 63), (20, 10, 64), (19, 10, 65), (22, 1, 17), (9, 1000, 33),
                                                   (640, 5, 40), (641, 320, 40), (1281, 7, 20), (2561, 40, 9),
                                                   (4096, 4095, 3), (4096, 1, 3)])
def test_make_pairs_regions(oracle, walk_len, window, walks):
    from paper_2407_15452_amd import binding as gs
    rng = np.random.default_rng(walk_len + window)
    w = rng.integers(0, 1 << 30, (walks, walk_len)).astype(np.int32)
    for i in range(walks):                                  # every valid length near the edges occurs
        keep = (walk_len, i % (walk_len + 1), min(walk_len, 2 * window + i % 3))[i % 3]
        w[i, keep:] = -1
    want_c, want_o = oracle.make_pairs(w, window)
    c, o, n = gs.gs_make_pairs(torch.as_tensor(w).to(DEV), window)
    assert n == want_c.size
    np.testing.assert_array_equal(c.cpu().numpy(), want_c)
    np.testing.assert_array_equal(o.cpu().numpy(), want_o)
