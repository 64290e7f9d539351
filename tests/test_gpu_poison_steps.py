"""The poison pass examines the launches that a run takes: on D2Q9 those of several steps.  The
launches are counted in a captured graph; poisoned ones feed one another and equal the oracle."""
import ctypes

import numpy as np
import pytest

from oracle import lattice as olat
from paper_2212_07494_amd import inputs
from tests.helpers import exact_mismatch, gpu_available, oracle_for

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a HIP device")]

TAU = (0.58, 0.87, 1.0)


def _hip():
    import torch  # noqa: F401  (its HIP runtime serves the library)
    with open("/proc/self/maps") as fh:
        path = next(m.split()[-1] for m in fh if "libamdhip64" in m)
    return ctypes.CDLL(path)


def _launches(stream, fn):
    """Nodes of the graph that fn() records on the stream (nothing runs)."""
    hip, graph, n = _hip(), ctypes.c_void_p(), ctypes.c_size_t()
    handle = ctypes.c_void_p(stream.cuda_stream)
    thread_local = 1
    assert hip.hipStreamBeginCapture(handle, thread_local) == 0
    fn()
    assert hip.hipStreamEndCapture(handle, ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    assert hip.hipGraphDestroy(graph) == 0
    return n.value


@pytest.mark.parametrize("poison", [False, True])
def test_launches_of_several_steps(poison):
    """32 x 32 FP64 takes seven steps a launch; each launch is preceded by a fill."""
    import torch
    from paper_2212_07494_amd import lbm as L
    stream = torch.cuda.Stream()
    with L.Lattice("D2Q9", "smrt", "f64", (32, 32, 1), (0, 0, 0), TAU, stream=stream,
                   debug_poison=poison) as lat:
        lat.step(7)
        stream.synchronize()
        assert _launches(stream, lambda: lat.step(15)) == 3 * (1 + poison)  # 7 + 7 + 1


@pytest.mark.parametrize("shape,walls,solid", [
    ((32, 32, 1), (0, 0, 0), False), ((64, 32, 1), (0, 1, 0), False), ((70, 47, 1), (1, 1, 0), True),
    ((130, 90, 1), (0, 0, 0), True), ((57, 5, 1), (0, 0, 0), False)])
def test_poisoned_launches_feed_one_another(shape, walls, solid):
    from paper_2212_07494_amd import lbm as L
    N, steps = int(np.prod(shape)), 23
    rng = np.random.default_rng(N)
    w = np.array([float(x) for x in olat.weights("D2Q9")])
    g = rng.uniform(-1e-3, 1e-3, (3, N))
    g[2] = 0
    mask = (rng.random(N) < 0.12).astype(np.uint8) if solid else None
    fluid = slice(None) if mask is None else mask == 0
    f0 = inputs.random_state(9, N, 5, scale=0.05, weights=w)
    o = oracle_for("D2Q9", "smrt", "f64", shape, walls, TAU)
    if solid:
        o = type(o)("D2Q9", "smrt", shape, walls=walls, tau=TAU, solid=mask)
    want = o.run(f0.copy(), g, steps)
    with L.Lattice("D2Q9", "smrt", "f64", shape, walls, TAU, g_field=g, solid=mask,
                   debug_poison=True) as lat:
        lat.set_populations(f0)
        lat.step(steps)
        assert exact_mismatch(lat.populations()[:, fluid], want[:, fluid]) == 0
