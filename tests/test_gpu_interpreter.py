"""The evaluation kernel's instruction streams and interpreter where they can
go wrong, bit for bit against the oracle: programs at the edges of an
instruction block (63 instructions and a reload), at the longest the
wavefront-parallel compiler takes (1,024 nodes) and beyond it, trees that
fill every register slot and reach into LDS, operands evaluated in either
order, constant subtrees, inputs the common paths leave to the caller; in
every launch configuration, on ragged rows."""
import os

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

NT = min(16, os.cpu_count() or 1)
N = oracle.node
CONFIGS = [(r, f, t, w) for r, f, t, w in ((1, 0, 1, 4), (1, 2, 3, 1), (2, 0, 2, 2), (2, 8, 1, 4), (4, 0, 1, 4), (4, 2, 2, 4),
                                           (4, 8, 1, 2), (1, 8, 2, 4), (2, 2, 1, 1))]


@pytest.fixture(scope="module")
def gp():
    import torch
    import paper_2110_11226_amd as gp
    torch.cuda.set_device(0)
    yield gp
    gp.set_launch_config(None)


def check(gp, progs, X, configs=CONFIGS):
    import torch
    op = oracle.from_programs(progs)
    host = gp.HostPopulation(op.nodes, op.prog_off, op.consts, op.const_off, op.length)
    gp.validate_population(host, X.shape[0])
    ref = oracle.evaluate_f32(op, X, n_threads=NT)
    pop = gp.DevicePopulation(host, n_features=X.shape[0])
    data = gp.DeviceDataset(X)
    for cfg in configs:
        if cfg[1] and X.shape[0] > cfg[1]:
            continue
        gp.set_launch_config(cfg)
        got = gp.evaluate(pop, data)
        torch.cuda.synchronize()
        got = got.cpu().numpy()
        same = (got.view(np.uint32) == ref.view(np.uint32)) | (np.isnan(got) & np.isnan(ref))
        assert same.all(), (cfg, np.argwhere(~same)[:3].tolist(), int((~same).sum()))
    gp.set_launch_config(None)


def rows(F, n, seed):
    return np.random.default_rng(seed).uniform(-4, 4, size=(F, n)).astype(np.float32)


def chain(n_un, op=8):
    return [N(op)] * n_un + [N(oracle.VAR, 0)], []


def fold(n_bin, F, rng):
    """n_bin binary functions, each with a terminal as one operand (its second
    at most 15 times: each of those holds a stack entry of the right-to-left
    scan)."""
    nodes, second = [N(oracle.VAR, 0)], 0
    for _ in range(n_bin):
        f = int(rng.integers(2, 6))
        term = [N(oracle.VAR, int(rng.integers(0, F)))]
        last = second < 15 and rng.random() < 0.5
        second += last
        nodes = [N(f)] + (nodes + term if last else term + nodes)
    return nodes, []


def full(depth, F, rng):
    if depth == 0:
        return [N(oracle.VAR, int(rng.integers(0, F)))]
    return [N(int(rng.integers(2, 6)))] + full(depth - 1, F, rng) + full(depth - 1, F, rng)


@pytest.mark.parametrize("F", [2, 5])
def test_instruction_block_edges(gp, F):
    rng = np.random.default_rng(1)
    lens = [0, 1, 60, 61, 62, 63, 64, 124, 125, 126, 127, 188, 189]
    progs = [chain(n) for n in lens] + [fold(n, F, rng) for n in lens]
    for n in (1, 63, 64, 257, 1000):
        check(gp, progs, rows(F, n, n))


@pytest.mark.parametrize("F", [2, 3])
def test_longest_parallel_programs_and_longer(gp, F):
    rng = np.random.default_rng(2)
    progs = [chain(n, 6) for n in (1021, 1022, 1023, 1024, 1300)]
    progs += [fold(n, F, rng) for n in (510, 511, 512, 700)]
    check(gp, progs, rows(F, 130, 3))


@pytest.mark.parametrize("depth", [1, 2, 8, 9, 10, 12])
def test_deep_trees(gp, depth):
    # depth 9 is the deepest full tree of the parallel path; from depth 10 the
    # right-to-left order holds depth + 1 entries, past the register slots
    rng = np.random.default_rng(depth)
    for F in (2, 6):
        check(gp, [(full(depth, F, rng), []) for _ in range(3)], rows(F, 300, depth))


def test_operand_orders_and_constants(gp):
    """Every binary function over all pairs of operand shapes: feature,
    constant, unary of each, a binary function, and one that needs more
    entries than the other operand."""
    v0, v1, c = [N(oracle.VAR, 0)], [N(oracle.VAR, 1)], "c"
    add = [N(oracle.ADD)]
    shapes = [v0, v1, [c], [N(9)] + v0, [N(9), c], add + v0 + v1, add + [c] + v1, add + [c, c],
              add + [N(10)] + v0 + [N(9)] + v1, add + add + [N(10)] + v0 + [N(9)] + v1 + add + [N(8)] + v0 + [N(7)] + v1]
    progs = []
    rng = np.random.default_rng(5)
    for f in (2, 3, 4, 5, 12, 13):
        for a in shapes:
            for b in shapes:
                nodes, consts = [], []
                for w in [N(f)] + a + b:
                    if isinstance(w, str):
                        nodes.append(N(oracle.CONST, len(consts)))
                        consts.append(float(np.float32(rng.uniform(-2, 2))))
                    else:
                        nodes.append(w)
                progs.append((nodes, consts))
    check(gp, progs, rows(2, 70, 6))


def test_inputs_left_to_the_caller(gp):
    """sin and cos from 2^24 on, logs of infinity, and NaN, on some rows of a
    lane only; and the same operations inside longer programs, between feature
    fetches, at the last instruction of a block."""
    x = rows(3, 300, 7)
    x[0, ::7] *= 1e9
    x[0, 3::11] = np.inf
    x[1, 5::13] = np.nan
    x[1, ::17] = -0.0
    un = [9, 10, 7, 8]
    progs = [([N(u), N(oracle.VAR, f)], []) for u in un for f in (0, 1)]
    progs += [([N(oracle.ADD), N(u)] + [N(oracle.MUL), N(oracle.VAR, 0), N(oracle.VAR, 0), N(oracle.VAR, 2)], []) for u in un]
    for n in (60, 61, 62):
        progs += [([N(6)] * n + [N(u), N(oracle.VAR, 0)], []) for u in un]
        progs += [([N(u)] + [N(6)] * n + [N(oracle.VAR, 0)], []) for u in un]
    check(gp, progs, x)


@pytest.mark.parametrize("P,n,cfg", [(1, 100_003, (1, 2, 1, 4)), (5000, 70, (1, 2, 1, 1)), (9, 4357, (4, 2, 1, 4)),
                                     (700, 20_011, (1, 2, 1, 4)), (3000, 2100, (1, 2, 1, 2)), (8, 2049, (4, 2, 64, 4))])
def test_work_claims(gp, P, n, cfg):
    """Fewer items than wavefronts, one chunk in one queue, more items than first
    claims cover, several items a claim: every item done once."""
    import torch
    host = gp.build_population(P, 2, "rhh", min_depth=1, max_depth=3, seed=P)
    X = rows(2, n, P)
    y = np.random.default_rng(1).normal(size=n).astype(np.float32)
    gp.set_launch_config(cfg)
    try:
        pop, data = gp.DevicePopulation(host, n_features=2), gp.DeviceDataset(X, y)
        out = gp.evaluate(pop, data)
        fit = [gp.fitness(pop, data, "mse").clone() for _ in range(2)]
        torch.cuda.synchronize()
    finally:
        gp.set_launch_config(None)
    op = oracle.Population(host.nodes, host.prog_off, host.consts, host.const_off, host.length)
    ref = oracle.evaluate_f32(op, X, n_threads=NT)
    got = out.cpu().numpy()
    same = (got.view(np.uint32) == ref.view(np.uint32)) | (np.isnan(got) & np.isnan(ref))
    assert same.all()
    assert torch.equal(fit[0], fit[1])
    with np.errstate(over="ignore", invalid="ignore"):
        want = ((ref.astype(np.float64) - y) ** 2).mean(axis=1).astype(np.float32)
    g = fit[0].cpu().numpy()
    fin = np.isfinite(want)
    assert np.array_equal(np.isfinite(g), fin)
    assert np.allclose(g[fin], want[fin], rtol=1e-6, atol=0)


def test_max_min_inverse_on_special_values(gp):
    """max, min and the protected inverse over every pair of signed zeros,
    NaN, infinities, denormals, the protection threshold and its neighbours."""
    eps = np.float32(0.001)
    v = np.array([0.0, -0.0, np.nan, np.inf, -np.inf, 1e-40, -1e-40, eps, -eps, np.nextafter(eps, np.float32(1)),
                  np.nextafter(eps, np.float32(0)), 1.0, -1.0, 3.4e38, 3e38, 2.9e38], np.float32)
    x = np.stack([np.repeat(v, len(v)), np.tile(v, len(v))])
    v0, v1 = N(oracle.VAR, 0), N(oracle.VAR, 1)
    progs = [([N(op), a, b], []) for op in (oracle.MAX, oracle.MIN) for a, b in ((v0, v1), (v1, v0))]
    # operands from a slot of the stack
    progs += [([N(op), N(oracle.NEG), v0, N(oracle.NEG), v1], []) for op in (oracle.MAX, oracle.MIN)]
    progs += [([N(oracle.INV), v0], []), ([N(oracle.NEG), N(oracle.INV), N(oracle.NEG), v0], [])]
    check(gp, progs, np.ascontiguousarray(x.astype(np.float32)))
