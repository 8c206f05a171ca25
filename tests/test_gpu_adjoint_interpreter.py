"""The adjoint's instruction streams and interpreter where they can go wrong,
against the oracle's reverse mode taken at the float32 evaluation: programs at
the edges of an instruction block, tapes that end in each of their three tiers
(26 entries in registers, 16 in LDS, then memory), constants summed in
registers (8), in LDS (16) and by atomics, the longest programs of the parallel
compiler (1,024 nodes) and one beyond it, operands of every shape in both
orders, inputs the common paths leave to the caller; on ragged rows, at every
number of rows per lane.

The tolerance is tests/test_gpu_adjoint.py's: 1e-4 of the derivative, 10 times
its Monte Carlo spread, 1e-6 of the program's largest."""
import numpy as np
import pytest

import oracle
from test_gpu_adjoint import check_grads, gp, oracle_reference, run_backward  # noqa: F401 (gp is a fixture)

pytestmark = pytest.mark.gpu
N = oracle.node
VALUES = (0.5, -1.25, 2.0, 0.75)


def program(words):
    """(nodes, consts) of a list of node words and "c" for a constant."""
    nodes, consts = [], []
    for w in words:
        if w == "c":
            nodes.append(N(oracle.CONST, len(consts)))
            consts.append(VALUES[len(consts) % len(VALUES)])
        else:
            nodes.append(w)
    return nodes, consts


def var(f=0):
    return N(oracle.VAR, f)


def unit(F, n, seed):
    """Magnitudes of 0.9 to 1.1: long products stay in range."""
    rng = np.random.default_rng(seed)
    return (rng.uniform(0.9, 1.1, size=(F, n)) * rng.choice([-1, 1], size=(F, n))).astype(np.float32)


def edge_programs():
    progs = []
    for n in (1, 12, 13, 14, 20, 21, 22, 25, 26, 27, 41, 42, 43, 60, 61, 62, 63, 64, 126, 128):
        progs.append([N(oracle.MUL), var(n % 2)] * n + ["c"])            # n entries, one constant
        progs.append([N(oracle.SIN)] * n + ["c"])
        progs.append([N(oracle.MUL)] + [N(oracle.NEG)] * n + ["c", var()])
        progs.append([N(oracle.ADD), "c"] * n + [var()])                 # n constants, no entry
    for n in (3, 7, 8, 9, 15, 16, 17, 30):
        progs.append(([N(oracle.ADD), N(oracle.MUL), "c", var()] * n + ["c"]))
        # two entries for each product of two subtrees with constants
        progs.append([N(oracle.MUL), N(oracle.ADD), "c", var()] * n + [var(1)])
        progs.append([N(oracle.DIV), N(oracle.ADD), "c", N(oracle.NEG), var()] * n + ["c"])
    return [program(p) for p in progs]


def order_programs():
    add = [N(oracle.ADD)]
    shapes = [[var()], ["c"], [N(oracle.SIN), "c"], [N(oracle.COS), var(1)], add + ["c", var()], add + [var(), var(1)],
              [N(oracle.MUL), "c", "c"], add + [N(oracle.SIN), var(), N(oracle.COS), "c"],
              add + add + [N(oracle.SIN), "c", N(oracle.COS), var()] + [N(oracle.MUL), "c", N(oracle.LOG), var(1)]]
    fs = (oracle.ADD, oracle.SUB, oracle.MUL, oracle.DIV, oracle.MAX, oracle.MIN, oracle.ATAN2)
    return [program([N(f)] + a + b) for f in fs for a in shapes for b in shapes]


def rare_programs():
    mul = [N(oracle.MUL), "c", var()]
    progs = []
    for u in (oracle.SIN, oracle.COS, oracle.LOG, oracle.SQRT, oracle.ABS, oracle.INV, oracle.SQ):
        progs += [[N(u)] + mul, [N(oracle.MUL), N(u)] + mul + [var(1)], [N(oracle.ADD), var(1), N(u)] + mul]
        progs += [[N(oracle.NEG)] * n + [N(u)] + mul for n in (59, 60, 61)]
    return [program(p) for p in progs]


def length_programs(longest):
    return [program([N(oracle.NEG)] * (n - 3) + [N(oracle.MUL), "c", var()]) for n in (longest - 2, longest - 1, longest)] + \
        [program(([N(oracle.MUL), N(oracle.NEG), var()] * 1000)[:longest - longest % 3 - 3] + ["c"])]


def case(name):
    if name == "edges":
        return edge_programs(), unit(2, 4099, 1), (1, 63, 65, 257, 4099)
    if name == "orders":
        return order_programs(), np.random.default_rng(2).uniform(0.3, 3, size=(2, 700)).astype(np.float32), (1, 700)
    if name == "rare":
        x = np.random.default_rng(3).uniform(-4, 4, size=(2, 1000)).astype(np.float32)
        x[0, ::37] *= np.float32(2.0 ** 24)
        x[0, 5::41] = 0.0
        x[0, 7::43] = 5e-4
        return rare_programs(), x, (64, 1000)
    return length_programs(int(name)), unit(2, 300, 4), (300,)


CASES = ("edges", "orders", "rare", "1024", "1025")


@pytest.mark.parametrize("rows", [0, 1, 2, 4])
@pytest.mark.parametrize("name", CASES)
def test_against_reverse_mode(gp, name, rows):  # noqa: F811
    progs, X, counts = case(name)
    op = oracle.from_programs(progs)
    host = gp.HostPopulation(op.nodes, op.prog_off, op.consts, op.const_off, op.length)
    gp.validate_population(host, 2)
    gp.set_launch_config((rows, 0, 1) if rows else None)
    try:
        for n in counts:
            x = np.ascontiguousarray(X[:, :n])
            y = np.random.default_rng(n).uniform(8, 12, size=n).astype(np.float32)
            print(f"adjoint: {name}, {n} rows, {rows} per lane", flush=True)
            g, _, _ = run_backward(gp, host, x, y, None, "mse", 2)
            g2, _, _ = run_backward(gp, host, x, y, None, "mse", 2)
            ref, spread, cond = oracle_reference(op, x, y, None, "mse")
            _, escaped = check_grads(host, g, ref, spread, cond, f"{name} {n} R={rows}")
            assert escaped == 0
            # the first sixteen constants are summed in a fixed order
            for p in range(host.n_programs):
                a, b = int(host.const_off[p]), int(host.const_off[p + 1])
                assert np.array_equal(g[a:min(b, a + 16)], g2[a:min(b, a + 16)])
    finally:
        gp.set_launch_config(None)
