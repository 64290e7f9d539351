"""Repeated read-backs: the first are copied, later small ones are written into pinned memory.
Each equals, bit for bit, what a lattice that is read once returns, on both sides of the
largest pinned size, with steps between the reads; monitors and batch domains likewise."""
import numpy as np
import pytest

from tests.helpers import gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a HIP device")]


def lattice(L, lat, shape):
    N = int(np.prod(shape))
    D = 2 if lat == "D2Q9" else 3
    rng = np.random.default_rng(3)
    return L.Lattice(lat, "smrt", "f64", shape, (0, 1, 0), (0.7, 0.9, 1.0), g=(1e-6, 0, 0),
                     rho=1 + 0.01 * rng.random(N), u=0.02 * rng.random((D, N)))


# 24 bytes a node on D2Q9: 257 x 170 is the last size of 1 MiB or less, 331 x 132 the first above
@pytest.mark.parametrize("lat,shape", [("D2Q9", (1, 3, 1)), ("D2Q9", (257, 170, 1)),
                                       ("D2Q9", (331, 132, 1)), ("D3Q19", (20, 7, 5))])
def test_repeated_reads(lat, shape):
    from paper_2212_07494_amd import lbm as L
    many = lattice(L, lat, shape)
    for k in range(12):
        once = lattice(L, lat, shape)
        if k:
            once.step(k)
            many.step(1)
        for a, b in zip(many.moments(), once.moments()):
            assert np.array_equal(a, b), k
        once.close()
    once = lattice(L, lat, shape)
    once.step(11)
    a, b = many.monitors(), once.monitors()
    assert a.mass == b.mass and list(a.mom) == list(b.mom) and list(a.j) == list(b.j)
    assert a.umax == b.umax and a.nonfinite == b.nonfinite == 0
    once.close()
    many.close()


def test_batch_reads_of_uneven_domains():
    from paper_2212_07494_amd import lbm as L
    doms = [dict(shape=s, walls=(0, 1, 0), tau=(0.7, 0.9, 1.0), g=(1e-6, 0, 0))
            for s in [(30, 9, 1), (100, 60, 1), (331, 132, 1), (257, 170, 1)]]
    with L.Batch(doms, "D2Q9", "smrt", "f64") as b:
        b.advance(6)
        first = [b.moments(d) for d in range(4)]   # all copied
        for _ in range(3):
            for d in (3, 0, 2, 1):
                for x, y in zip(b.moments(d), first[d]):
                    assert np.array_equal(x, y), d
