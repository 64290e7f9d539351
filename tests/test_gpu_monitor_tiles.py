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
