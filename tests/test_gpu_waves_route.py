"""lbm_set_waves where a node sums its own waves (narrow rows, few waves) and where its row's
are summed, against the sum as written; and rows whose blocks would pass the largest launch."""
import math

import numpy as np
import pytest

from oracle import lattice as olat
from tests.helpers import gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a HIP device")]


def _check(lat, shape, nw, nodes=None, solid=None, storage="f64"):
    from paper_2212_07494_amd import lbm as L
    L.load()
    nx, ny, nz = shape
    w = np.array([olat.to_f64(v) for v in olat.weights(lat)])
    rng = np.random.default_rng(nw + nx)
    k = rng.integers(-2 * nx, 2 * nx + 1, size=(nw, 3)).astype(np.int32)
    k[0] = (nx // 2, ny // 2, nz // 2)
    phase = rng.uniform(-7.0, 7.0, size=nw)
    amp = (rng.normal(size=(nw, w.size)) + 1j * rng.normal(size=(nw, w.size))) * 1e-3
    n = np.arange(nx * ny * nz) if nodes is None else np.asarray(nodes)
    c = (n % nx, (n // nx) % ny, n // (nx * ny))
    want = np.repeat(w[:, None], n.size, axis=1)
    for kw, ph, a in zip(k.astype(np.int64), phase, amp):
        th = 2 * math.pi * sum((kw[d] * c[d] % shape[d]) / shape[d] for d in range(3)) + ph
        want += np.outer(a.real, np.cos(th)) - np.outer(a.imag, np.sin(th))
    # each wave's angle and factors to a few units of roundoff on either side, and the sums'
    tol = 2.0 ** -53 * (40 * np.abs(amp).sum() / w.size * 4 + nw * np.abs(want).max())
    if storage == "f16s":  # and a deviation's rounding to binary16
        tol += 2.0 ** -11 * np.abs(want - w[:, None]).max()
    with L.Lattice(lat, "smrt", storage, shape, (0, 0, 0), (0.8, 1.0, 1.0), solid=solid) as lt:
        lt.set_waves(k, phase, amp)
        got = lt.populations(nodes) + (w[:, None] if storage == "f16s" else 0)
        live = slice(None) if solid is None else solid == 0
        np.testing.assert_allclose(got[:, live], want[:, live], rtol=0, atol=tol)


@pytest.mark.parametrize("lat,shape,nw", [
    ("D2Q9", (1, 300, 1), 7), ("D2Q9", (130, 9, 1), 1), ("D3Q19", (5, 70, 3), 185),
    ("D3Q27", (16, 9, 11), 185), ("D3Q27", (17, 9, 11), 20), ("D3Q39", (129, 5, 3), 4),
    ("D3Q27", (64, 5, 3), 60), ("D3Q19", (3, 2, 2), 2)])
def test_routes(lat, shape, nw):
    _check(lat, shape, nw)


def test_solid_nodes_by_node():
    """Pulls from solid nodes bounce back: the slots of the solid nodes' neighbours."""
    shape = (7, 30, 4)
    solid = (np.random.default_rng(2).random(7 * 30 * 4) < 0.1).astype(np.uint8)
    _check("D3Q19", shape, 5, solid=solid)


def test_rows_beyond_the_largest_launch():
    """8192^2 rows of one node: four rows a workgroup of 256 threads would be 2^32 threads."""
    n = 8192
    nodes = np.array([0, 1, 255, 256, n, n * n // 2 + 3, n * n - n, n * n - 2, n * n - 1])
    _check("D3Q19", (1, n, n), 3, nodes=nodes, storage="f16s")
