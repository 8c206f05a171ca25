"""Genetic operations with a wavefront per offspring, word for word against the
oracle: each operation alone on parents whose lengths lie at the edges of the
64 nodes a wavefront takes at a time, offspring counts on both sides of every
spread of the donors over wavefronts, and length bounds that force hoisting
through long donors."""
import numpy as np
import pytest

import oracle
from test_gpu_mutate import _lib_init, _oracle_pop, _same, gp  # noqa: F401 (gp is a fixture)

pytestmark = pytest.mark.gpu
LENGTHS = (1, 2, 3, 62, 63, 64, 65, 66, 127, 128, 129, 130, 191, 192, 193, 260)


def parents(gp, seed):  # noqa: F811
    progs = []
    for n in LENGTHS:
        h = gp.build_population(3, 3, "exact_len", min_len=n, max_len=n, max_consts=0, seed=seed + n)
        for p in range(3):
            a, b = int(h.prog_off[p]), int(h.prog_off[p + 1])
            c, d = int(h.const_off[p]), int(h.const_off[p + 1])
            progs.append((h.nodes[a:b], h.consts[c:d]))
    op = oracle.from_programs(progs)
    return gp.HostPopulation(op.nodes, op.prog_off, op.consts, op.const_off, op.length)


def reference(host, init, ev, n_off, generation):
    e = oracle.EvolveParams(**ev)
    ops, first, T = oracle.plan_generation(e, n_off, generation)
    win = np.random.default_rng(n_off).integers(0, host.n_programs, size=T).astype(np.int32)
    return ops, first, win, oracle.mutate(e, oracle.InitParams(**init), _oracle_pop(host), ops, first, win, generation)


def compare(gp, host, init, ev, n_off, generation):  # noqa: F811
    ops, first, win, ref = reference(host, init, ev, n_off, generation)
    d_ops, d_first, _ = gp.plan_generation_device(n_off, generation, **ev)
    assert np.array_equal(d_ops.cpu().numpy(), ops) and np.array_equal(d_first.cpu().numpy(), first)
    off = gp.mutate_device(gp.DevicePopulation(host, n_features=3), d_ops, d_first, win, generation, _lib_init(init), **ev)
    _same(off.to_host(), ref, (n_off, generation, ev))


@pytest.mark.parametrize("op", ["p_crossover", "p_subtree", "p_hoist", "p_point", None])
@pytest.mark.parametrize("max_len", [40, 400])
def test_each_operation_at_wavefront_edges(gp, op, max_len):  # noqa: F811
    host = parents(gp, 5)
    ev = dict(p_crossover=0.0, p_subtree=0.0, p_hoist=0.0, p_point=0.0, p_point_replace=0.4, max_len=max_len, seed=31)
    if op:
        ev[op] = 1.0
    init = dict(n_features=3, method="exact_len", min_depth=1, max_depth=3, min_len=1, max_len=200, max_consts=0)
    compare(gp, host, init, ev, 700, 4)


@pytest.mark.parametrize("n_off", [1, 3, 4, 5, 511, 512, 1023, 1024, 2048, 4096, 8191, 8192, 16384])
def test_counts_around_each_spread(gp, n_off):  # noqa: F811
    host = parents(gp, 6)
    ev = dict(p_crossover=0.3, p_subtree=0.4, p_hoist=0.1, p_point=0.1, p_point_replace=0.3, max_len=300, seed=32)
    init = dict(n_features=3, method="rhh", min_depth=1, max_depth=4, min_len=1, max_len=50, max_consts=4)
    compare(gp, host, init, ev, n_off, 2)
