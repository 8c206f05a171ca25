"""The backward pass's log-loss is gp_fitness's: on one row, where there is no
summation order to differ in, fitness_out has gp_fitness's very bits, for the
kernel of programs up to 1,024 nodes at each number of rows per lane and for
that of longer ones."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("negs,P", [(0, 30_000), (1024, 3000)])
@pytest.mark.parametrize("R", [1, 2, 4])
def test_one_row(negs, P, R):
    import torch
    import paper_2110_11226_amd as gp
    rng = np.random.default_rng(3 + negs)
    a = np.concatenate([rng.integers(0x32000000, 0x42d20000, size=P - 8).astype(np.uint32).view(np.float32),
                        np.array([0.0, 1e-38, 88.0, 103.9, 104.0, 150.0, 200.0, 3e38], np.float32)])
    a[::2] *= -1.0
    L = negs + 1
    one = [oracle.node(oracle.NEG)] * negs + [oracle.node(oracle.CONST, 0)]
    off = np.arange(P + 1, dtype=np.int64)
    host = gp.HostPopulation(np.tile(np.array(one, np.uint32), P), off * L, a, off, np.full(P, L, np.int32))
    pop = gp.DevicePopulation(host, n_features=1)
    for label in (0.0, 1.0):
        data = gp.DeviceDataset(np.zeros((1, 1), np.float32), np.full(1, label, np.float32))
        print(f"log-loss backward: {L} nodes, {R} rows per lane, label {label}", flush=True)
        gp.set_launch_config((R, 0, 1, 4))
        try:
            want = gp.fitness(pop, data, "logloss")
            got = torch.empty(P, dtype=torch.float32, device="cuda")
            gp.fitness_backward(pop, data, "logloss", fitness_out=got)
            torch.cuda.synchronize()
        finally:
            gp.set_launch_config(None)
        want, got = want.cpu().numpy(), got.cpu().numpy()
        assert np.array_equal(got.view(np.uint32), want.view(np.uint32)), int((got != want).sum())
