"""Tournaments over several lanes, winner for winner against the oracle: sizes
around a block of four draws and a whole wavefront of blocks, counts on both
sides of every number of lanes, ties, NaN and signed zeros among the draws."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P", [1, 3, 700])
@pytest.mark.parametrize("metric", ["mse", "pearson"])
def test_sizes_ties_and_nan(P, metric):
    import torch
    import paper_2110_11226_amd as gp
    rng = np.random.default_rng(P)
    ln = rng.integers(1, 4, size=P).astype(np.int32)
    for kind in ("ties", "nan", "all nan"):
        fit = rng.integers(-1, 2, size=P).astype(np.float32) * np.float32(0.0 if kind == "ties" else 0.5)
        if kind != "ties":
            fit[rng.random(P) < (0.6 if kind == "nan" else 2.0)] = np.nan
        for k in (1, 4, 5, 8, 9, 16, 17, 33, 64, 65, 128, 129, 255, 256, 257, 1030):
            for T in (1, 63, 513):
                for c in (0.0, 0.25):
                    win = gp.tournament(torch.from_numpy(fit).cuda(), torch.from_numpy(ln).cuda(), metric, c, k, T, k, 1)
                    ref = oracle.tournament(fit, ln, gp.larger_is_better(metric), c, k, T, k, 1)
                    assert np.array_equal(win.cpu().numpy(), ref), (kind, k, T, c)


@pytest.mark.parametrize("lanes", [1, 2, 4, 8, 16])
def test_counts_around_each_number_of_lanes(lanes):
    import torch
    import paper_2110_11226_amd as gp
    rng = np.random.default_rng(lanes)
    P = 501
    fit = rng.integers(0, 20, size=P).astype(np.float32)
    ln = rng.integers(1, 9, size=P).astype(np.int32)
    for T in (131072 // lanes, 131072 // lanes + 1):
        win = gp.tournament(torch.from_numpy(fit).cuda(), torch.from_numpy(ln).cuda(), "mse", 0.5, 70, T, 4, 2)
        ref = oracle.tournament(fit, ln, False, 0.5, 70, T, 4, 2)
        assert np.array_equal(win.cpu().numpy(), ref), T
