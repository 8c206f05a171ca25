"""Programs of more than 1,024 nodes and the others take different kernels of
the backward pass, each by its own length: a program's gradient and fitness
are the same bits whatever bound max_len gives, and whatever programs are in
the population beside it."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

CFG = (4, 0, 2, 4)


@pytest.fixture(scope="module")
def gp():
    import torch
    import paper_2110_11226_amd as gp
    torch.cuda.set_device(0)
    yield gp
    gp.set_launch_config(None)


def join(gp, hosts):
    at, ct = np.cumsum([0] + [h.prog_off[-1] for h in hosts]), np.cumsum([0] + [h.const_off[-1] for h in hosts])
    return gp.HostPopulation(np.concatenate([h.nodes for h in hosts]),
                             np.concatenate([[0]] + [h.prog_off[1:] + a for h, a in zip(hosts, at)]).astype(np.int64),
                             np.concatenate([h.consts for h in hosts]),
                             np.concatenate([[0]] + [h.const_off[1:] + c for h, c in zip(hosts, ct)]).astype(np.int64),
                             np.concatenate([h.length for h in hosts]))


def backward(gp, host, data, metric, max_len=None):
    import torch
    pop = gp.DevicePopulation(host, n_features=2)
    if max_len:
        pop.view.max_len = max_len
    fit = torch.full((host.n_programs,), 7.0, dtype=torch.float32, device="cuda")
    grad = gp.fitness_backward(pop, data, metric, fitness_out=fit)
    torch.cuda.synchronize()
    return grad.cpu().numpy().view(np.uint32), fit.cpu().numpy().view(np.uint32)


@pytest.mark.parametrize("metric", ["mae", "mse", "rmse", "logloss", "pearson"])
def test_by_length(gp, metric):
    N = 1500
    rng = np.random.default_rng(3)
    X = rng.uniform(-2, 2, size=(2, N)).astype(np.float32)
    y = (rng.random(N) < 0.5).astype(np.float32) if metric == "logloss" else (X[0] * X[1]).astype(np.float32)
    data = gp.DeviceDataset(X, y)

    def build(P, lo, hi, seed):      # (16 constants: further slots are summed in no fixed order)
        return gp.build_population(P, 2, "exact_len", min_len=lo, max_len=hi, max_consts=16, seed=seed)
    parts = [build(50, 1, 60, 1), build(3, 1025, 1025, 2), build(3, 1020, 1024, 3), build(9, 1025, 1600, 4), build(40, 1, 200, 5)]
    gp.set_launch_config(CFG)
    try:
        alone = [backward(gp, h, data, metric) for h in parts]
        for max_len in (1025, 4096):
            print(f"{metric}: short programs, bound {max_len}", flush=True)
            g, f = backward(gp, parts[0], data, metric, max_len)
            assert np.array_equal(g, alone[0][0]) and np.array_equal(f, alone[0][1])
        for order in ((0, 1, 2, 3, 4), (3, 4), (1, 0), (2, 1), (1, 3)):
            print(f"{metric}: parts {order}", flush=True)
            g, f = backward(gp, join(gp, [parts[k] for k in order]), data, metric)
            assert np.array_equal(g, np.concatenate([alone[k][0] for k in order]))
            assert np.array_equal(f, np.concatenate([alone[k][1] for k in order]))
    finally:
        gp.set_launch_config(None)
