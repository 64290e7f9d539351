"""Ragged widths: the block shape 64 x 3 takes consecutive nodes, 64 x 2 rows.  Single steps of
both, in every addressing path, against the oracle bit for bit; the tuner keeps one of them."""
import numpy as np
import pytest

from oracle import lattice as olat
from paper_2212_07494_amd import inputs
from tests.helpers import exact_mismatch, gpu_available, oracle_for, to_storage

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a HIP device")]

TAU = (0.58, 0.87, 1.0)


@pytest.mark.parametrize("lat,shape,walls,solid", [
    ("D3Q19", (1, 7, 5), (0, 0, 0), False), ("D3Q19", (3, 50, 4), (1, 0, 0), False),
    ("D3Q27", (65, 9, 4), (0, 1, 1), False), ("D3Q19", (131, 6, 5), (0, 1, 1), True),
    ("D3Q39", (70, 8, 5), (0, 0, 0), False), ("D2Q9", (100, 2, 1), (0, 0, 0), False),
    ("D2Q9", (100, 9, 1), (0, 1, 0), True), ("D2Q9", (1, 300, 1), (0, 0, 0), False),
    ("D3Q27", (90, 11, 3), (1, 1, 0), False), ("D3Q19", (67, 1, 3), (0, 0, 0), False)])
def test_consecutive_nodes_and_rows(lat, shape, walls, solid):
    from paper_2212_07494_amd import lbm as L
    L.load()
    N = int(np.prod(shape))
    rng = np.random.default_rng(N)
    w = np.array([float(x) for x in olat.weights(lat)])
    g = rng.uniform(-1e-3, 1e-3, (3, N))
    if lat == "D2Q9":
        g[2] = 0
    mask = (rng.uniform(0, 1, N) < 0.1).astype(np.uint8) if solid else None
    fluid = slice(None) if mask is None else mask == 0
    for storage in ("f64", "f32s", "f16s"):
        f0 = inputs.random_state(len(w), N, 3, scale=0.05, weights=w)
        f0 = to_storage(f0 - (w[:, None] if storage != "f64" else 0), storage)
        o = oracle_for(lat, "smrt", storage, shape, walls, TAU)
        if solid:
            o = type(o)(lat, "smrt", shape, walls=walls, tau=TAU, shift=o._p.shift, real=o.real,
                        store16=bool(o._p.store16), solid=mask)
        fo = o.run(f0.astype(o.dtype), g, 2).astype(np.float64)
        with L.Lattice(lat, "smrt", storage, shape, walls, TAU, g_field=g, solid=mask) as gpu:
            for bx, by, v in [(64, 3, 0), (64, 3, 4), (64, 3, 9), (64, 3, 14), (64, 3, 59),
                              (64, 2, 0), (64, 2, 4), (64, 2, 9), (64, 2, 38)]:
                gpu.tune(bx, by, v)
                gpu.set_populations(f0)
                gpu.step(1)
                gpu.step(1)
                assert exact_mismatch(gpu.populations()[:, fluid], fo[:, fluid]) == 0, (bx, by, v)


@pytest.mark.parametrize("steps", [1, 3, 20])
def test_tuner_keeps_the_state(steps):
    from paper_2212_07494_amd import lbm as L
    shape = (90, 20, 12)
    rng = np.random.default_rng(1)
    with L.Lattice("D3Q19", "smrt", "f32s", shape, (0, 1, 0), TAU, g=(1e-5, 0, 0),
                   u=0.02 * rng.random((3, 90 * 20 * 12))) as lat:
        lat.step(3)
        f = lat.populations()
        t, ms = L.lbm_autotune(lat.ctx, steps)
        assert ms > 0 and lat.tune() == t and lat.time == 3
        assert exact_mismatch(lat.populations(), f) == 0
