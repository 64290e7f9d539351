"""Single steps on widths that fill no wavefront (blocks of consecutive nodes), against the
oracle bit for bit: every addressing path and block size, walls across each axis (rows that
may and may not bounce back), solid nodes, widths from one node up, layers that end inside a
block; and the quotient the blocks' rows come from."""
import numpy as np
import pytest

from oracle import lattice as olat
from paper_2212_07494_amd import inputs
from tests.helpers import exact_mismatch, gpu_available, oracle_for, to_storage

TAU = (0.58, 0.87, 1.0)


def test_division_by_multiplication():
    """n // nx = (n m) >> (31 + s) with m = ceil(2^(31+s) / nx), for n < 2^31."""
    rng = np.random.default_rng(1)
    for nx in [2, 3, 5, 63, 65, 127, 131, 1000, 65537, 2 ** 30 - 1, 2 ** 30 + 1, 2 ** 31 - 1]:
        s = (nx - 1).bit_length()
        m = ((1 << (31 + s)) + nx - 1) // nx
        assert m < 1 << 32
        n = [0, nx - 1, nx, 2 ** 31 - 1, 2 ** 31 - 2]
        n += [int(q) * nx + d for q in rng.integers(1, max(2, 2 ** 31 // nx), 200) for d in (-1, 0)]
        for v in n:
            if 0 <= v < 2 ** 31:
                assert ((v * m) >> 32) >> (s - 1) == v // nx, (nx, v)


@pytest.mark.gpu
@pytest.mark.skipif(not gpu_available(), reason="needs a HIP device")
@pytest.mark.parametrize("lat,shape,walls,solid", [
    ("D3Q19", (1, 7, 5), (0, 0, 0), False), ("D3Q19", (3, 50, 4), (1, 0, 0), False),
    ("D3Q27", (65, 9, 4), (0, 1, 1), False), ("D3Q19", (131, 6, 5), (0, 1, 1), True),
    ("D3Q39", (70, 8, 5), (0, 0, 0), False), ("D2Q9", (100, 2, 1), (0, 0, 0), False),
    ("D3Q27", (90, 11, 3), (1, 1, 0), False), ("D3Q19", (67, 1, 3), (0, 0, 0), False)])
def test_linear_blocks(lat, shape, walls, solid):
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
    for storage in ("f64", "f32s"):
        f0 = inputs.random_state(len(w), N, 3, scale=0.05, weights=w)
        f0 = to_storage(f0 - (w[:, None] if storage == "f32s" else 0), storage)
        o = oracle_for(lat, "smrt", storage, shape, walls, TAU)
        if solid:
            o = type(o)(lat, "smrt", shape, walls=walls, tau=TAU, shift=o._p.shift, real=o.real,
                        store16=bool(o._p.store16), solid=mask)
        fo = o.run(f0.astype(o.dtype), g, 2).astype(np.float64)
        with L.Lattice(lat, "smrt", storage, shape, walls, TAU, g_field=g, solid=mask) as gpu:
            # 64 x 2 takes consecutive nodes on these widths, the others rows
            for bx, by, v in [(64, 2, 0), (64, 2, 4), (64, 2, 9), (64, 2, 14), (64, 1, 0),
                              (64, 4, 4), (128, 2, 8), (256, 1, 9), (128, 1, 10)]:
                gpu.tune(bx, by, v)
                gpu.set_populations(f0)
                gpu.step(2)
                assert exact_mismatch(gpu.populations()[:, fluid], fo[:, fluid]) == 0, (bx, by, v)
