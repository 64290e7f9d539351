"""64-bit addressing with bounce-back: population buffers just above 4 GiB, with walls, in
blocks of rows and of consecutive nodes, at sampled nodes beside the walls and in the last
layers; and the same lattice just below, whose offsets fit 32 bits."""
import numpy as np
import pytest

from tests.helpers import gpu_available, oracle_for
from tests.test_gpu_parity import _sampled_step_parity

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a HIP device")]


# 27 x 8 bytes a node: 4 GiB is 19,884,107 nodes; 259 columns fill no wavefront, 256 do
@pytest.mark.parametrize("shape,above", [((259, 277, 281), True), ((259, 277, 277), False),
                                         ((256, 280, 281), True)])
def test_walled_buffers_at_4gib(shape, above):
    from paper_2212_07494_amd import lbm as L
    nx, ny, nz = shape
    N = nx * ny * nz
    assert (27 * 8 * N >= 1 << 32) == above
    walls, tau = (1, 0, 1), (0.7, 1.0, 1.0)
    table = np.zeros((3, nx))
    table[0] = 1e-4 * np.cos(0.1 * np.arange(nx))
    table[1] = 2e-4 * np.sin(0.3 * np.arange(nx))
    rng = np.random.default_rng(1)
    nodes = np.unique(np.concatenate([
        [0, nx - 1, N - nx, N - 1, nx * ny - 1, N - nx * ny],         # corners of the walls
        N - 1 - rng.integers(0, nx * ny, 60),                         # last layer
        rng.integers(0, nx * ny, 40),                                 # first layer
        rng.integers(0, ny * nz, 60) * nx,                            # beside the walls of x
        rng.integers(0, ny * nz, 60) * nx + nx - 1,
        rng.integers(0, N, 80)]))
    o = oracle_for("D3Q27", "smrt", "f64", shape, walls, tau)
    g = np.zeros((3, N))  # only the sampled nodes' entries are read
    g[:, nodes] = table[:, nodes % nx]
    with L.Lattice("D3Q27", "smrt", "f64", shape, walls, tau, g_profile=(0, table)) as gpu:
        gpu.step(2)
        for t in ((64, 3, 0), (64, 3, 4), (64, 4, 0), (256, 1, 4)):
            gpu.tune(*t)
            assert _sampled_step_parity(gpu, o, "D3Q27", shape, walls, g, nodes, "f64") == 0, t
