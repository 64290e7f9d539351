"""Replayed chunks of lattices that take several steps a launch: a chunk of 50 x 200 D2Q9 is 70
steps, so calls of 140 steps or more replay."""
import math

import numpy as np
import pytest

from tests.helpers import exact_mismatch, gpu_available

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs a HIP device")]

ARGS = ("D2Q9", "smrt")
KW = dict(g=(-1e-4, 0.0, 0.0))
SHAPE = ((50, 200, 1), (0, 1, 0), (0.8, 1.0, 1.0))


@pytest.mark.parametrize("storage", ["f64", "f32s"])
def test_replays_equal_direct_launches(storage):
    """Calls of two chunks and a remainder, of one step less than two chunks, and of many,
    with eager work between them, against the same steps in pieces too short to replay."""
    from paper_2212_07494_amd import lbm as L
    s = np.cos(2 * math.pi * np.arange(1000) / 1200)
    with L.Lattice(*ARGS, storage, *SHAPE, **KW) as a, L.Lattice(*ARGS, storage, *SHAPE, **KW) as b:
        t = 0
        for n in (150, 139, 140, 330, 150):
            a.step(n, s[t:t + n])
            for i in range(0, n, 100):
                b.step(min(100, n - i), s[t + i:t + min(n, i + 100)])
            t += n
            assert a.time == b.time == t
            assert exact_mismatch(a.populations(), b.populations()) == 0, (n, t)
            a.moments()


def test_a_replaying_call_does_not_block():
    """Graphs, device and pinned staging are made by a first call of 150 steps (two chunks and
    a remainder); then 20,000 steps are enqueued while they run, and a second call that reuses
    the staging gives what one call of both gives."""
    import torch
    from paper_2212_07494_amd import lbm as L
    s = np.cos(2 * math.pi * np.arange(40_000) / 1200)
    stream = torch.cuda.Stream()
    with L.Lattice(*ARGS, "f64", *SHAPE, stream=stream, **KW) as a, \
            L.Lattice(*ARGS, "f64", *SHAPE, stream=stream, **KW) as b:
        a.step(150, s[:150])
        b.step(150, s[:150])
        stream.synchronize()
        a.step(20_000, s[150:20_150])
        pending = not stream.query()
        a.step(19_850, s[20_150:])
        b.step(39_850, s[150:])
        assert exact_mismatch(a.populations(), b.populations()) == 0
        assert pending
