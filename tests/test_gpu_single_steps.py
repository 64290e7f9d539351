"""Single steps of D2Q9, which longer calls take several a launch: taken a call each, in every
launch configuration (block shapes x variants x wave caps), with solid nodes, and in batches
over tile policies, persistent grids and memory variants, against the oracle bit for bit."""
import numpy as np
import pytest

from oracle import lattice as olat
from paper_2212_07494_amd import inputs
from tests.helpers import exact_mismatch, gpu_available, oracle_for, to_storage
from tests.test_gpu_batch import d2_domains, g_field_of
from tests.test_gpu_variants import CASES, TAU, VARIANTS

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a HIP device")]

W9 = np.array([float(x) for x in olat.weights("D2Q9")])


def _start(N, storage, seed, scale=None):
    kw = {} if scale is None else dict(scale=scale)
    f0 = inputs.random_state(9, N, seed, weights=W9, **kw)
    return to_storage(f0 - (W9[:, None] if storage != "f64" else 0), storage)


@pytest.mark.parametrize("storage", ["f64", "f32s", "f16s"])
@pytest.mark.parametrize("coll", ["bgk", "smrt", "rmrt"])
def test_all_launch_configurations(coll, storage):
    from paper_2212_07494_amd import lbm as L
    L.load()
    for shape, walls in CASES["D2Q9"]:
        N = int(np.prod(shape))
        f0 = _start(N, storage, 3)
        g = np.random.default_rng(4).uniform(-1e-3, 1e-3, (3, N))
        g[2] = 0
        o = oracle_for("D2Q9", coll, storage, shape, walls, TAU[coll])
        want = o.run(f0.astype(o.dtype), g, 3).astype(np.float64)
        with L.Lattice("D2Q9", coll, storage, shape, walls, TAU[coll], g_field=g) as gpu:
            for bx, by in ((64, 1), (64, 2), (64, 3), (64, 4), (128, 1), (128, 2), (256, 1)):
                for v in VARIANTS:
                    gpu.tune(bx, by, v)
                    gpu.set_populations(f0)
                    for _ in range(3):
                        gpu.step(1)
                    bad = exact_mismatch(gpu.populations(), want)
                    assert bad == 0, (shape, walls, bx, by, v, bad)


@pytest.mark.parametrize("storage", ["f64", "f32s", "f16s"])
@pytest.mark.parametrize("coll", ["bgk", "smrt", "rmrt"])
@pytest.mark.parametrize("walls", [(0, 0, 0), (0, 1, 0), (1, 1, 0)])
def test_solid_nodes(coll, storage, walls):
    from paper_2212_07494_amd import lbm as L
    shape = (70, 37, 1)
    N = 70 * 37
    rng = np.random.default_rng(17)
    solid = (rng.uniform(0, 1, N) < 0.15).astype(np.uint8)
    fluid = solid == 0
    g = rng.uniform(-1e-3, 1e-3, (3, N))
    g[2] = 0
    f0 = _start(N, storage, 19, 0.05)
    o = oracle_for("D2Q9", coll, storage, shape, walls, TAU[coll])
    o = type(o)("D2Q9", coll, shape, walls=walls, tau=TAU[coll], shift=o._p.shift, real=o.real,
                store16=bool(o._p.store16), solid=solid)
    scales = (1.0, 0.5, -2.0)
    fo = f0.astype(o.dtype)
    for s in scales:
        fo = o.step(fo, g, s)
    fo = fo.astype(np.float64)
    with L.Lattice("D2Q9", coll, storage, shape, walls, TAU[coll], g_field=g, solid=solid) as gpu:
        for t in (None, (64, 3, 0), (64, 2, 4), (256, 1, 9)):
            if t:
                gpu.tune(*t)
            gpu.set_populations(f0)
            for s in scales:
                gpu.step(1, g_scale=[s])
            assert exact_mismatch(gpu.populations()[:, fluid], fo[:, fluid]) == 0, t


@pytest.mark.parametrize("storage", ["f64", "f32s", "f16s"])
def test_batch_configurations(storage):
    from paper_2212_07494_amd import lbm as L
    _, doms = d2_domains(16, seed=3)
    doms.append(dict(shape=(5, 3, 1), walls=(1, 0, 0), tau=(0.7, 0.9, 1.0), g=(1e-5, 0, 0)))
    want = []
    for dom in doms:
        o = oracle_for("D2Q9", "smrt", storage, dom["shape"], dom["walls"], dom["tau"])
        g = g_field_of(dom)
        want.append(o.run(o.init(1.0, None, g), g, 5).astype(np.float64))
    with L.Batch(doms, "D2Q9", "smrt", storage) as b:
        start = [b.populations(d) for d in range(len(doms))]
        for tbx in (0, 1, 64, 128, 256):
            for bpc in (0, 1, 8):
                for v in (0, 1, 2):
                    b.tune(tbx, bpc, v)
                    for d, f in enumerate(start):
                        b.set_populations(d, f)
                    for _ in range(5):
                        b.advance(1)
                    for d in range(len(doms)):
                        assert exact_mismatch(b.populations(d), want[d]) == 0, (tbx, bpc, v, d)
