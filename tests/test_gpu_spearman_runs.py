"""Tied runs of the Spearman kernels where they can go wrong: runs that begin,
end or lie wholly at the edges of 64 positions and of a wavefront's range, on
either side, from all-distinct values to one run of every row.  Values are
small integers and products of two of them, exact on both sides, so the
oracle's fitness must come out to float32 rounding (1e-6 relative)."""
import os

import numpy as np
import pytest

import oracle
from test_gpu_spearman import gp, gpu_spearman  # noqa: F401 (gp is a fixture)

pytestmark = pytest.mark.gpu
NT = min(16, os.cpu_count() or 1)


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("N", [1, 2, 63, 64, 65, 128, 1023, 1024, 1025, 4097, 65_537, 140_000])
def test_runs(gp, N, weighted):  # noqa: F811
    rng = np.random.default_rng(N)
    V, C = oracle.node(oracle.VAR, 0), oracle.node(oracle.CONST, 0)

    def column(levels):
        """`levels` values in runs of about the same length, shuffled rows"""
        return rng.permutation(np.arange(N) * levels // N).astype(np.float32)
    levels = sorted({min(k, N) for k in (1, 2, 3, 17, 64, 1000, N)})
    cols = [column(k) for k in levels]
    # one long run between distinct values
    long_run = np.arange(N, dtype=np.float32)
    long_run[N // 5:N // 5 + max(1, N // 2)] = N // 5
    cols.append(rng.permutation(long_run))
    X = np.ascontiguousarray(np.stack(cols))
    w = rng.integers(1, 5, size=N).astype(np.float32) if weighted else None
    progs = [([oracle.node(oracle.VAR, f)], []) for f in range(len(cols))]
    progs += [([oracle.node(oracle.MUL), C, oracle.node(oracle.VAR, f)], [-0.5]) for f in range(len(cols))]
    progs += [([oracle.node(oracle.SUB), V, V], []), ([C], [3.0])]
    op = oracle.from_programs(progs)
    host = gp.HostPopulation(op.nodes, op.prog_off, op.consts, op.const_off, op.length)
    for y in (cols[0], cols[len(cols) // 2], cols[-2], cols[-1]):
        y = rng.permutation(y)
        got = gpu_spearman(gp, host, X, y, w, X.shape[0])
        ref, _ = oracle.fitness(op, X, y, w, "spearman", n_threads=NT)
        assert np.allclose(got, ref, rtol=1e-6, atol=1e-7, equal_nan=True), np.abs(got - ref).max()
