"""Programs of more than 1,024 nodes and the others take different kernels of
the backward pass, each by its own length: a program's gradient and fitness
are the same bits whatever bound max_len gives, and whatever programs are in
the population beside it."""
import numpy as np
import pytest

import oracle
from test_gpu_adjoint import check_grads, oracle_reference, run_backward
from test_gpu_adjoint_interpreter import program

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


def densest(units):
    """Quotients of `units` roots of constants: the most instructions for the
    nodes (6 a node)."""
    if units == 1:
        return [oracle.node(oracle.SQRT), "c"]
    return [oracle.node(oracle.DIV)] + densest((units + 1) // 2) + densest(units // 2)


def test_streams_that_fill_their_room(gp):
    """Next to each other, so that a word past a program's room would be in
    its neighbour's stream."""
    lists = [densest(u) for u in (1, 2, 3, 4, 8, 21, 64, 340, 341, 1, 341, 341, 2)]
    op = oracle.from_programs([program(w) for w in lists])
    assert op.length.max() == 1022
    host = gp.HostPopulation(op.nodes, op.prog_off, op.consts, op.const_off, op.length)
    X = np.random.default_rng(5).uniform(-1, 1, size=(2, 65)).astype(np.float32)
    y = np.random.default_rng(6).uniform(8, 12, size=65).astype(np.float32)
    for R in (1, 4):
        print(f"densest programs, {R} rows per lane", flush=True)
        gp.set_launch_config((R, 0, 1))
        try:
            g, _, _ = run_backward(gp, host, X, y, None, "mse", 2)
        finally:
            gp.set_launch_config(None)
        ref, spread, cond = oracle_reference(op, X, y, None, "mse")
        _, escaped = check_grads(host, g, ref, spread, cond, f"densest R={R}")
        assert escaped == 0
