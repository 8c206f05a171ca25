"""The log-loss's log(1 + e^-|z|) on the device, alone: a constant program z < 0
on one row of label 0 has it as its fitness.  It is formed in double to 2^-32
and rounded once, so it lies within 0.51 units in the last place (of a normal
float; the least denormal's below) of the float64 value."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def test_every_binade():
    import torch
    import paper_2110_11226_amd as gp
    rng = np.random.default_rng(1)
    u = np.concatenate([np.arange(0, 0x43480000, 40_009, dtype=np.uint32),                       # 0 .. 200
                        rng.integers(0x32000000, 0x42d20000, size=60_000).astype(np.uint32),     # 7e-9 .. 105
                        np.array([0x42cff1b5, 0x42ce8ed0, 0x42aeac50, 0x3f317218, 0x3f800000, 0x43480000, 0x7f7fffff,
                                  0x7f800000], np.uint32)])
    a = u.view(np.float32)
    P = a.size
    host = gp.HostPopulation(np.full(P, oracle.node(oracle.CONST, 0), np.uint32), np.arange(P + 1, dtype=np.int64), -a,
                             np.arange(P + 1, dtype=np.int64), np.ones(P, np.int32))
    pop = gp.DevicePopulation(host, n_features=1)
    data = gp.DeviceDataset(np.zeros((1, 1), np.float32), np.zeros(1, np.float32))
    got = gp.fitness(pop, data, "logloss")
    torch.cuda.synchronize()
    got = got.cpu().numpy().astype(np.float64)
    fin = np.isfinite(a)
    assert np.isnan(got[~fin]).all()                  # 0 times an infinite output
    a64 = a[fin].astype(np.float64)
    want = np.log1p(np.exp(-a64))
    ulp = np.maximum(np.spacing(want.astype(np.float32)).astype(np.float64), 2.0 ** -149)
    assert (np.abs(got[fin] - want) <= 0.51 * ulp).all(), float((np.abs(got[fin] - want) / ulp).max())
