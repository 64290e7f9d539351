"""The monitor pass over few tiles and over more tiles than it has blocks (2048)."""
import numpy as np
import pytest

from tests.helpers import gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a HIP device")]


def test_records_of_a_small_lattice():
    """A lattice holds as many block records as its smallest blocks could leave, no more."""
    from paper_2212_07494_amd import lbm as L
    with L.Lattice("D2Q9", "smrt", "f64", (70, 20, 1), (0, 1, 0), (0.7, 0.9, 1.0)) as lat:
        # two buffers, recorded velocities, the force, 2 x 20 block records and the record
        N = 70 * 20
        assert L.lbm_device_bytes(lat.ctx) <= 8 * (2 * 9 * N + 3 * N + 3 + (40 + 1) * 11) + 4096
        want = N
        for bx, by in ((64, 1), (128, 1), (64, 4), (256, 1)):
            lat.tune(bx, by, 0)
            lat.step(1)
            assert abs(lat.monitors().mass - want) < 1e-9


def _fields(rng, N, D):
    return 1 + 0.01 * rng.random(N), 0.02 * (rng.random((D, N)) - 0.5)


# at 64 x 1: 2 x 45 x 50 = 4500 tiles; 70 columns fill no wavefront, 45 rows no block of two
@pytest.mark.parametrize("storage", ["f64", "f32s"])
@pytest.mark.parametrize("lat,shape,walls,tune", [
    ("D3Q19", (70, 45, 50), (0, 1, 1), (64, 1, 0)), ("D3Q27", (130, 45, 31), (1, 0, 0), (128, 2, 4)),
    ("D3Q19", (70, 90, 50), (0, 0, 0), (64, 2, 9)), ("D2Q9", (301, 1999, 1), (0, 1, 0), (64, 4, 3))])
def test_blocks_walk_several_tiles(lat, shape, walls, tune, storage):
    """Mass, momenta, largest speed and residual against sums of the fields of both times."""
    from paper_2212_07494_amd import lbm as L
    N, D = int(np.prod(shape)), 2 if lat == "D2Q9" else 3
    rho, u = _fields(np.random.default_rng(5), N, D)
    g = (1e-5, -2e-5, 0.0)
    with L.Lattice(lat, "smrt", storage, shape, walls, (0.7, 0.9, 1.0), rho=rho, u=u, g=g) as gpu:
        gpu.tune(*tune)
        gpu.step(2)
        r0, u0 = gpu.moments()
        gpu.monitors()
        gpu.step(1)
        r, u = gpu.moments()
        m = gpu.monitors()
    # sums of N terms of either side in binary64: N roundings of the largest partial sum
    eps = 2.0 ** -53 * N
    assert m.nonfinite == 0 and m.step == 3
    assert abs(m.mass - r.sum()) <= eps * np.abs(r).sum()
    for c in range(D):
        assert abs(m.mom[c] - (r * u[c]).sum()) <= eps * np.abs(r * u[c]).sum()
        # rho u = j + rho g / 2 at each node, in the arithmetic type
        tiny = (2.0 ** -52 if storage == "f64" else 2.0 ** -23) * 8
        assert abs(m.j[c] - (r * (u[c] - g[c] / 2)).sum()) <= (eps + tiny) * np.abs(r * u[c]).sum()
    speed = np.sqrt((u * u).sum(0))
    assert abs(m.umax - speed.max()) <= 4 * 2.0 ** -53 * speed.max()
    du2, u2 = ((u - u0) ** 2).sum(), (u * u).sum()
    assert abs(m.resid - np.sqrt(du2 / u2)) <= 4 * eps * np.sqrt(du2 / u2)


@pytest.mark.parametrize("where", [0, 2047, 2048, 4499])
def test_a_late_tile_counts(where):
    """One NaN in the tile `where` of 4500 (64 x 1 blocks) is counted once, with its neighbours
    none: a population that the node pulls from itself (the rest population)."""
    from paper_2212_07494_amd import lbm as L
    shape = (70, 45, 50)
    nx, ny, _ = shape
    with L.Lattice("D3Q19", "smrt", "f64", shape, (0, 1, 1), (0.7, 0.9, 1.0)) as gpu:
        gpu.tune(64, 1, 0)
        f = gpu.populations()
        tx, row = where % 2, where // 2
        f[0, row * nx + 64 * tx + 3] = np.nan
        gpu.set_populations(f)
        assert gpu.monitors().nonfinite == 1
