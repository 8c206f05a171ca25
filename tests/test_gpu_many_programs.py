"""Jobs of fewer row chunks than work queues, whose programs are dealt to the
queues: every program on every chunk exactly once, whatever their number
(fewer than queues, not a multiple of them, far more than wavefronts)."""
import numpy as np
import pytest

import oracle
from _parity import check_rows_exact, to_oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gp():
    import torch
    import paper_2110_11226_amd as gp
    torch.cuda.set_device(0)
    yield gp
    gp.set_launch_config(None)


@pytest.mark.parametrize("P", [1, 7, 8, 9, 1001, 20_003])
@pytest.mark.parametrize("chunks", [1, 2, 7, 8, 9])
def test_every_program_on_every_chunk(gp, P, chunks):
    import torch
    N = 64 * chunks - 5
    X = np.random.default_rng(chunks).uniform(-3, 3, size=(2, N)).astype(np.float32)
    host = gp.build_population(P, 2, "exact_len", min_len=1, max_len=9, max_consts=4, seed=P)
    pop = gp.DevicePopulation(host, n_features=2)
    y = X[0] * X[1]
    data = gp.DeviceDataset(X, y)
    print(f"{P} programs, {chunks} chunks", flush=True)
    gp.set_launch_config((1, 2, 1, 4))
    try:
        out = torch.full((P, N), 7.0, dtype=torch.float32, device="cuda")
        gp.evaluate(pop, data, out=out)
        fit = gp.fitness(pop, data, "mae")
        bfit = torch.full((P,), 7.0, dtype=torch.float32, device="cuda")
        gp.fitness_backward(pop, data, "mae", fitness_out=bfit)
        torch.cuda.synchronize()
    finally:
        gp.set_launch_config(None)
    out, fit, bfit = out.cpu().numpy(), fit.cpu().numpy(), bfit.cpu().numpy()
    check_rows_exact(out, oracle.evaluate_f32(to_oracle(host), X, n_threads=8), f"{P} programs, {chunks} chunks")
    with np.errstate(all="ignore"):
        want = np.abs(out.astype(np.float64) - y.astype(np.float64)).mean(axis=1)
    for got in (fit, bfit):      # float64 sums of at most 571 non-negative terms, rounded once
        fin = np.isfinite(want)
        assert np.array_equal(np.isnan(got), np.isnan(want))
        assert (np.abs(got[fin] - want[fin]) <= (2.0 ** -24 + 1e-12) * want[fin] + 1e-45).all()
