"""sin and cos around 2^24, where the Payne-Hanek reduction takes over (and
around 2^20, well below), bit for bit against the oracle: every float next to
the switch, in both signs, and at every number of rows per lane, so that lanes
and rows on either side of it share a wavefront."""
import numpy as np
import pytest

from test_gpu_crmath import compare, gp, programs  # noqa: F401 (gp is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 2, 4])
@pytest.mark.parametrize("exponent", [20, 24, 25])
def test_around_the_switch(gp, rows, exponent):  # noqa: F811
    op, host = programs(gp)
    pop = gp.DevicePopulation(host, n_features=1)
    at = int(np.float32(2.0 ** exponent).view(np.uint32))
    near = np.arange(at - 300, at + 301, dtype=np.uint32)
    bits = np.concatenate([near, near | np.uint32(0x80000000), np.array([0x3f800000] * 7, np.uint32)])
    bits = np.random.default_rng(exponent).permutation(bits)
    gp.set_launch_config((rows, 0, 1, 4))
    try:
        compare(gp, op, pop, bits)
    finally:
        gp.set_launch_config(None)
