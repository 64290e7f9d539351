"""Small read-backs borrow pinned memory of the process: from the first read on they take no
device memory; more lattices, threads and sizes than there are blocks (8 of 1 MiB) read what a
copy from the device returns; lattices opened and closed in between."""
import threading

import numpy as np
import pytest

from tests.helpers import gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a HIP device")]


def _lattice(L, shape, seed, stream=None):
    N = int(np.prod(shape))
    rng = np.random.default_rng(seed)
    return L.Lattice("D2Q9", "smrt", "f64", shape, (0, 1, 0), (0.7, 0.9, 1.0), g=(1e-6, 0, 0),
                     rho=1 + 0.01 * rng.random(N), u=0.02 * rng.random((2, N)), stream=stream)


def _equal(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a, b))


def test_first_small_read_takes_no_device_memory():
    from paper_2212_07494_amd import lbm as L
    with L.Lattice("D2Q9", "smrt", "f64", (30, 20, 1), (0, 1, 0), (0.7, 0.9, 1.0)) as lat:
        before = L.lbm_device_bytes(lat.ctx)
        lat.moments()
        lat.monitors()
        assert L.lbm_device_bytes(lat.ctx) == before


def test_many_lattices_in_turn():
    from paper_2212_07494_amd import lbm as L
    shapes = [(16 + 7 * k, 9 + k, 1) for k in range(20)] + [(400, 200, 1)]  # the last is copied
    lats = [_lattice(L, s, k) for k, s in enumerate(shapes)]
    first = [lat.moments() for lat in lats]
    for k in range(0, len(lats), 3):  # closing gives nothing away that others read
        lats[k].close()
        lats[k] = _lattice(L, shapes[k], k)
    assert all(_equal(lat.moments(), f) for lat, f in zip(lats, first))
    for lat in lats:
        lat.close()


def test_threads_and_streams():
    """Twelve threads, each its lattice and stream, step and read at once."""
    import torch
    from paper_2212_07494_amd import lbm as L
    n, rounds = 12, 25
    want = []
    for k in range(n):
        with _lattice(L, (20 + 11 * k, 30, 1), k) as lat:
            reads = []
            for _ in range(rounds):
                lat.step(3)
                reads.append(lat.moments())
            want.append((reads, lat.monitors().mass))
    bad, streams = [], [torch.cuda.Stream() for _ in range(n)]

    def work(k):
        try:
            with _lattice(L, (20 + 11 * k, 30, 1), k, streams[k]) as lat:
                for r in range(rounds):
                    lat.step(3)
                    if not _equal(lat.moments(), want[k][0][r]):
                        bad.append((k, r))
                if lat.monitors().mass != want[k][1]:
                    bad.append((k, "mass"))
        except Exception as e:  # reported by the assertion below
            bad.append((k, repr(e)))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(n)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
    assert not bad
