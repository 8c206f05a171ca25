"""User functions on a deep stack, on the GPU, bit for bit against the
oracle: runs of calls that fill their room of the instruction stream to the
last word, between short programs whose streams lie next to theirs, and
definitions of a single node."""
import os

import numpy as np
import pytest

import oracle
from _parity import check_fitness_exact, check_rows_exact, to_oracle

pytestmark = pytest.mark.gpu

n = oracle.node
A, B, C = n(oracle.VAR, 0), n(oracle.VAR, 1), n(oracle.CONST, 0)
X0, X1 = n(oracle.VAR, 0), n(oracle.VAR, 1)
U1, U2 = oracle.USER1, oracle.USER2
DEEP = [n(oracle.ADD)] * 12
CASES = {
    "argument plus constant": {U1: ([n(oracle.ADD), A, C], [0.5])},
    "single nodes": {U1: ([A], []), U1 + 1: ([C], [0.25]), U2: ([A], []), U2 + 1: ([B], [])},
    "both orders": {U1: ([n(oracle.SUB), C, A], [0.5]), U2: ([n(oracle.SUB), B, A], []), U2 + 1: ([n(oracle.DIV), A, B], [])},
}


@pytest.mark.parametrize("case", list(CASES))
def test_long_runs_of_calls_between_short_programs(case):
    import torch
    import paper_2110_11226_amd as gp
    defs = CASES[case]
    for op, (d, c) in defs.items():
        gp.register_function(op, d, c)
        oracle.set_user_function(op, d, c)
    try:
        def run(op, calls, deep):
            binary = op >= U2
            return ((DEEP if deep else []) + sum(([n(op)] + ([X1] if binary else []) for _ in range(calls)), [])
                    + [X0] + ([X1] * 12 if deep else []), [])
        short = [([n(oracle.SUB), X0, X1], []), ([n(oracle.SIN), X1], []), ([X0], [])]
        progs = []
        for op in defs:
            for calls in (1, 63, 1500, 4000):
                for deep in (False, True):
                    progs += [run(op, calls, deep)] + short
        pop = oracle.from_programs(progs)
        host = gp.HostPopulation(pop.nodes, pop.prog_off, pop.consts, pop.const_off, pop.length)
        X = np.random.default_rng(8).uniform(-2, 2, size=(2, 300)).astype(np.float32)
        dev = gp.DevicePopulation(host, n_features=2)
        data = gp.DeviceDataset(X)
        ref = oracle.evaluate_f32(to_oracle(host), X, n_threads=min(16, os.cpu_count() or 1))
        for cfg in ((4, 2, 1, 4), (1, 0, 1, 4)):
            print(f"calls: {case} {cfg}", flush=True)
            gp.set_launch_config(cfg)
            out = gp.evaluate(dev, data)
            torch.cuda.synchronize()
            check_rows_exact(out.cpu().numpy(), ref, f"{case} {cfg}")
    finally:
        gp.set_launch_config(None)
        for op in defs:
            gp.register_function(op)
            oracle.set_user_function(op)


@pytest.mark.parametrize("P,max_len", [(3073, 60), (6200, 30), (20_003, 20), (200_003, 4)])
@pytest.mark.parametrize("loss", [False, True])
def test_groups_of_programs(P, max_len, loss):
    """With user functions about, a compiling wavefront takes a group of
    programs (one up to 3,072 programs on 256 CUs, 60 from 181,000 on), some
    left to a lane each: those with calls, one of more than 1,024 nodes, one
    deeper than the register slots; the last group is not full."""
    import torch
    import paper_2110_11226_amd as gp
    defs = {U1: ([n(oracle.MUL), A, A], []), U2: ([n(oracle.SUB), n(oracle.MUL), A, B, C], [0.5]),
            U2 + 3: ([n(oracle.MUL), n(oracle.SUB), A, B, n(oracle.SUB), A, B], [])}
    mask = oracle.DEFAULT_FMASK | (1 << U1) | (1 << U2)
    for op, (d, c) in defs.items():
        gp.register_function(op, d, c)
        oracle.set_user_function(op, d, c)
    try:
        host = gp.build_population(P - 2, 2, "exact_len", min_len=1, max_len=max_len, max_consts=4, function_mask=mask, seed=9)
        extra = [([n(oracle.SQRT)] * 1100 + [X0], []), ([n(oracle.ADD)] * 18 + [X0] + [X1] * 18, [])]
        tail = oracle.from_programs(extra)
        host = gp.HostPopulation(np.concatenate([host.nodes, tail.nodes]),
                                 np.concatenate([host.prog_off, host.prog_off[-1] + tail.prog_off[1:]]), host.consts,
                                 np.concatenate([host.const_off, np.full(2, host.const_off[-1])]),
                                 np.concatenate([host.length, tail.length]))
        N = 40
        X = np.random.default_rng(4).uniform(-2, 2, size=(2, N)).astype(np.float32)
        y = X[0] - X[1]
        dev, data = gp.DevicePopulation(host, n_features=2), gp.DeviceDataset(X, y)
        print(f"groups: {P} programs, loss {loss}", flush=True)
        if loss:
            got = gp.fitness(dev, data, "user3")
            torch.cuda.synchronize()
            f32p, f64 = oracle.fitness(to_oracle(host), X, y, None, "user3", n_threads=min(16, os.cpu_count() or 1))
            check_fitness_exact(got.cpu().numpy(), f32p, f64, label=f"groups {P}")
        else:
            out = gp.evaluate(dev, data)
            torch.cuda.synchronize()
            ref = oracle.evaluate_f32(to_oracle(host), X, n_threads=min(16, os.cpu_count() or 1))
            check_rows_exact(out.cpu().numpy(), ref, f"groups {P}")
    finally:
        for op in defs:
            gp.register_function(op)
            oracle.set_user_function(op)
