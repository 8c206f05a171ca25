"""The largest shapes the launch heuristic has to leave room for: partial sums
that fit gp_fitness_noalloc's 64 MiB array (16,777,216 rows x 4,096 programs
among them) and work items below 2^30."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def aligned(n):
    return (n + 255) // 256 * 256


def chunks(gp, F, N, P, metric):
    R, _, tiles, _ = gp.get_launch_config(F, N, P, metric)
    return -(-N // (tiles * 64 * R))


def noalloc_bytes(P, nodes, C, metric):
    k = 4 if metric == "pearson" else 1
    return 1024 + 2 * aligned(4 * P) + aligned(16 * (nodes + 1)) + aligned(8 * P * C * k) + aligned(32 * C)


@pytest.fixture(scope="module")
def gp():
    import torch
    import paper_2110_11226_amd as gp
    torch.cuda.set_device(0)
    gp.set_launch_config(None)
    gp.autotune_clear()
    return gp


@pytest.mark.parametrize("N,P,mean,metric", [(16_777_216, 4096, 100, "mse"), (16_777_216, 4096, 100, "logloss"),
                                             (16_777_216, 1024, 100, "pearson"), (1_048_576, 65_536, 15, "mae")])
def test_partial_sums_fit_the_static_array(gp, N, P, mean, metric):
    C = chunks(gp, 2, N, P, metric)
    assert noalloc_bytes(P, mean * P, C, metric) <= 64 << 20, C


@pytest.mark.parametrize("metric", ["mae", "mse", "logloss", "pearson"])
def test_work_items_stay_below_their_bound(gp, metric):
    for N, P in ((16_800_000, 300_000), (16_777_216, 1_000_000), (1_048_576, 16_000_000)):
        assert chunks(gp, 2, N, P, metric) * P <= 1 << 30, (N, P)


def test_fitness_without_allocation_at_16M_rows_by_4096_programs(gp):
    import torch
    N, P = 16_777_216, 4096
    g = torch.Generator(device="cuda").manual_seed(1)
    data = gp.DeviceDataset(torch.rand((2, N), generator=g, device="cuda"), torch.rand(N, generator=g, device="cuda"))
    pop = gp.DevicePopulation(gp.build_population(P, 2, "exact_len", min_len=1, max_len=3, seed=5), n_features=2)
    got, want = gp.fitness_noalloc(pop, data, "mse"), gp.fitness(pop, data, "mse")
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy().view(np.uint32), want.cpu().numpy().view(np.uint32))


def test_longer_chunks_beside_many_nodes(gp):
    """Streams that leave too little of the array for the heuristic's chunks."""
    import torch
    N, P, L = 1_048_576, 8192, 400
    assert noalloc_bytes(P, L * P, chunks(gp, 3, N, P, "mse"), "mse") > 64 << 20
    g = torch.Generator(device="cuda").manual_seed(2)
    data = gp.DeviceDataset(torch.rand((3, N), generator=g, device="cuda"), torch.rand(N, generator=g, device="cuda"))
    pop = gp.DevicePopulation(gp.build_population(P, 3, "exact_len", min_len=L, max_len=L, seed=6), n_features=3)
    got, want = gp.fitness_noalloc(pop, data, "mse"), gp.fitness(pop, data, "mse")
    torch.cuda.synchronize()
    # sums of squares in another order: within N 2^-53 of each other, 1e-10, so
    # that the float32 results are at most neighbours
    got, want = (x.cpu().numpy().view(np.int32).astype(np.int64) for x in (got, want))
    assert np.abs(got - want).max() <= 1


@pytest.mark.parametrize("F,N,P,metric,tiles", [(28, 11_000_000, 2000, "logloss", 16), (28, 16_777_216, 1024, "pearson", 16),
                                                (5, 16_777_216, 1000, "pearson", 48), (2, 16_777_216, 4096, "mse", 48)])
def test_chunks_no_longer_than_the_partial_sums_ask_for(gp, F, N, P, metric, tiles):
    """A chunk of many features that is longer than the programs share in an L2
    takes up to a third more time."""
    R, _, t, _ = gp.get_launch_config(F, N, P, metric)
    assert R == 4 and t <= tiles


def test_many_features_without_allocation(gp):
    """Partial sums of 128 MiB at the launch's own chunks."""
    import torch
    F, N, P = 28, 4_194_304, 4096
    assert noalloc_bytes(P, 3 * P, chunks(gp, F, N, P, "pearson"), "pearson") > 64 << 20
    g = torch.Generator(device="cuda").manual_seed(7)
    data = gp.DeviceDataset(torch.rand((F, N), generator=g, device="cuda"), torch.rand(N, generator=g, device="cuda"))
    pop = gp.DevicePopulation(gp.build_population(P, F, "exact_len", min_len=1, max_len=3, seed=8), n_features=F)
    got, want = gp.fitness_noalloc(pop, data, "pearson"), gp.fitness(pop, data, "pearson")
    torch.cuda.synchronize()
    got, want = got.cpu().numpy().astype(np.float64), want.cpu().numpy().astype(np.float64)
    # moments in another order: their float64 sums within N 2^-53 of each other
    # relative to sums of absolute terms, the correlation within 1e-9 and a rounding
    assert np.array_equal(np.isnan(got), np.isnan(want))
    assert np.nanmax(np.abs(got - want)) <= 1e-9 + 2.0 ** -23


def test_a_device_resident_run_holds_no_adjoint_stream(gp):
    """Its memory: two populations (8 bytes a node of capacity each) and the
    evaluation's stream (16), the rest within 128 MiB."""
    import torch
    P, max_len = 8192, 2048
    cap = P * max_len
    init = dict(n_features=2, method="rhh", min_depth=2, max_depth=4)
    host = gp.build_population(P, 2, "rhh", min_depth=2, max_depth=4, seed=1)
    data = gp.DeviceDataset(np.zeros((2, 64), np.float32), np.ones(64, np.float32))
    gp.tournament(gp.fitness(gp.DevicePopulation(host, n_features=2), data), torch.ones(P, dtype=torch.int32, device="cuda"))
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    evo = gp.Evolution(data, host, init, dict(max_len=max_len), max_generations=2)
    evo.run(1)
    held = before - torch.cuda.mem_get_info()[0]
    evo.close()
    print(f"held {held / cap:.2f} bytes a node of capacity", flush=True)
    assert held <= 32 * cap + (128 << 20)


def test_the_autotuner_stays_within_the_longest_chunks(gp):
    """It times a prefix of 1,048,576 rows, on which longer chunks than any the
    heuristic takes look better than they are for the whole."""
    import torch
    N, P = 16_777_216, 4096
    pop = gp.DevicePopulation(gp.build_population(P, 2, method="exact_len", min_len=1, max_len=20, seed=3), n_features=2)
    X = torch.zeros(2, N, device="cuda")
    data = gp.DeviceDataset(X, torch.zeros(N, device="cuda"))
    try:
        (R, _, tiles, _), ms = gp.autotune(pop, data, "mse", repeats=1)
    finally:
        gp.autotune_clear()
    assert ms > 0.0 and R * tiles <= 4 * 64, (R, tiles)
