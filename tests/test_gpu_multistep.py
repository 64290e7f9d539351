"""Several steps a launch on D2Q9 (tiles with recomputed margins) against the oracle, bit for
bit: widths on both sides of a tile of 64 columns and of two tiles, heights from the fewest
rows up, remainders of the steps of a launch, every storage, collision, wall and force kind,
solid nodes, replayed graphs, and batches that mix such domains."""
import numpy as np
import pytest

from oracle import lattice as olat
from paper_2212_07494_amd import inputs
from tests.helpers import exact_mismatch, gpu_available, oracle_for, to_storage

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a HIP device")]

W9 = np.array([float(x) for x in olat.weights("D2Q9")])
TAU = (0.58, 0.87, 1.0)


def lbm():
    from paper_2212_07494_amd import lbm as L
    L.load()
    return L


def _force(kind, shape, rng):
    """(Lattice arguments, (3, N) field)"""
    nx, ny, _ = shape
    N = nx * ny
    if kind == "field":
        g = rng.uniform(-1e-3, 1e-3, (3, N))
        g[2] = 0
        return dict(g_field=g), g
    if kind == "uniform":
        v = rng.uniform(-1e-3, 1e-3, 3) * [1, 1, 0]
        return dict(g=v), np.repeat(v[:, None], N, 1)
    axis = 0 if kind == "x" else 1
    t = rng.uniform(-1e-3, 1e-3, (3, shape[axis]))
    t[2] = 0
    return dict(g_profile=(axis, t)), inputs.profile_field(shape, axis, t)


CASES = [
    # nx, ny, walls, force, steps, collision, storage, options
    (64, 12, (0, 0, 0), "y", 5, "smrt", "f64", {}),
    (65, 13, (0, 0, 0), "field", 11, "smrt", "f32s", {}),
    (63, 12, (0, 0, 0), "x", 7, "bgk", "f16s", {}),
    (57, 3, (0, 0, 0), "y", 4, "smrt", "f64", {}),
    (113, 11, (0, 0, 0), "uniform", 9, "rmrt", "f32", {}),
    (1, 5, (0, 1, 0), "y", 5, "bgk", "f64", {}),
    (2, 1, (0, 1, 0), "uniform", 6, "smrt", "f64", {}),
    (66, 2, (0, 1, 0), "field", 5, "smrt", "f32s", {}),
    (64, 40, (1, 1, 0), "x", 8, "bgk", "f64", {}),
    (130, 61, (1, 0, 0), "y", 5, "smrt", "f32s", {}),
    (129, 300, (1, 1, 0), "field", 5, "rmrt", "f64", {}),
    (300, 333, (0, 0, 0), "field", 6, "smrt", "f16s", {}),
    (40, 14, (0, 0, 0), "field", 7, "smrt", "f64", {}),
    (32, 33, (0, 1, 0), "y", 14, "bgk", "f64", {}),
    (33, 3, (1, 1, 0), "x", 13, "smrt", "f32s", {}),
    (70, 37, (0, 0, 0), "y", 5, "smrt", "f64", dict(force_order=3)),
    (70, 37, (0, 1, 0), "y", 5, "smrt", "f32s", dict(force_order=4)),
    (70, 37, (0, 0, 0), "field", 5, "smrt", "f64", dict(tau_bulk=0.9)),
]


@pytest.mark.parametrize("nx,ny,walls,force,steps,coll,storage,options", CASES)
def test_multistep_matches_oracle(nx, ny, walls, force, steps, coll, storage, options):
    L = lbm()
    shape, N = (nx, ny, 1), nx * ny
    rng = np.random.default_rng(nx + 1000 * ny)
    kw, g = _force(force, shape, rng)
    f0 = inputs.random_state(9, N, 5, scale=0.05, weights=W9)
    f0 = to_storage(f0 - (W9[:, None] if storage.endswith("s") else 0), storage)
    o = oracle_for("D2Q9", coll, storage, shape, walls, TAU, **options)
    scales = 1.0 + 0.5 * np.sin(np.arange(steps))
    with L.Lattice("D2Q9", coll, storage, shape, walls, TAU, **kw, **options) as gpu:
        gpu.set_populations(f0)
        gpu.step(steps, g_scale=scales)
        assert gpu.time == steps
        fo = f0.astype(o.dtype)
        for s in scales:
            fo = o.step(fo, g, s)
        assert exact_mismatch(gpu.populations(), fo.astype(np.float64)) == 0


@pytest.mark.parametrize("walls", [(0, 0, 0), (0, 1, 0), (1, 1, 0)])
@pytest.mark.parametrize("nx,ny", [(64, 20), (150, 47)])
def test_multistep_solid_nodes(nx, ny, walls):
    L = lbm()
    shape, N = (nx, ny, 1), nx * ny
    rng = np.random.default_rng(3)
    solid = (rng.uniform(0, 1, N) < 0.15).astype(np.uint8)
    kw, g = _force("field", shape, rng)
    f0 = to_storage(inputs.random_state(9, N, 5, scale=0.05, weights=W9), "f64")
    o = oracle_for("D2Q9", "smrt", "f64", shape, walls, TAU)
    o = type(o)("D2Q9", "smrt", shape, walls=walls, tau=TAU, solid=solid)
    with L.Lattice("D2Q9", "smrt", "f64", shape, walls, TAU, solid=solid, **kw) as gpu:
        gpu.set_populations(f0)
        gpu.step(8)
        fo = o.run(f0.copy(), g, 8)
        fluid = solid == 0
        assert exact_mismatch(gpu.populations()[:, fluid], fo[:, fluid]) == 0


@pytest.mark.parametrize("steps", [139, 140, 213])
def test_multistep_graphs(steps):
    """Replayed chunks with and without factors, twice, with eager steps between."""
    L = lbm()
    shape = (50, 33, 1)
    rng = np.random.default_rng(9)
    kw, g = _force("y", shape, rng)
    s = np.cos(0.1 * np.arange(steps))
    o = oracle_for("D2Q9", "smrt", "f64", shape, (0, 1, 0), TAU)
    with L.Lattice("D2Q9", "smrt", "f64", shape, (0, 1, 0), TAU, **kw) as gpu:
        f = gpu.populations()
        for _ in range(2):
            gpu.step(steps, g_scale=s)
            gpu.step(3)
            gpu.step(steps)
            for v in s:
                f = o.step(f, g, v)
            f = o.run(f, g, 3 + steps)
            assert exact_mismatch(gpu.populations(), f) == 0


@pytest.mark.parametrize("coll,storage,rows", [("smrt", "f64", 12), ("bgk", "f32s", 12),
                                               ("smrt", "f32s", 5), ("smrt", "f64", 2)])
def test_multistep_batch(coll, storage, rows):
    """Domains around the tile edges; `rows` rows in the lowest periodic one (12: launches of
    five steps, 5: of three, 2: none)."""
    L = lbm()
    rng = np.random.default_rng(rows)
    shapes = [((64, rows, 1), (0, 0, 0), "y"), ((65, 30, 1), (0, 0, 0), "field"),
              ((20, 16, 1), (0, 1, 0), "uniform"), ((130, 64, 1), (1, 1, 0), "x"),
              ((7, 2, 1), (0, 1, 0), "uniform"), ((200, 97, 1), (1, 0, 0), "y")]
    doms, fields = [], []
    for shape, walls, kind in shapes:
        kw, g = _force(kind, shape, rng)
        doms.append(dict(shape=shape, walls=walls, tau=TAU, **kw))
        fields.append(g)
    with L.Batch(doms, "D2Q9", coll, storage) as b:
        b.advance(9)
        b.run(12, 0.0, check_every=6, stall_checks=100)
        for d, (dom, g) in enumerate(zip(doms, fields)):
            o = oracle_for("D2Q9", coll, storage, dom["shape"], dom["walls"], TAU)
            fo = o.run(o.init(1.0, None, g), g, 21)
            assert exact_mismatch(b.populations(d), fo.astype(np.float64)) == 0, d
