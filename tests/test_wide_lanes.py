"""Bunches whose lanes lie on both sides of the short series' bounds in most waves:
the oracle's results, and a time that shows that a wave does not run a second body
for the lanes beyond them.
"""

import math

import numpy as np
import pytest

import oracle
from test_parity_fp64 import assert_parity, gpu_run
from workloads import Beam, gaussian_bunch, rhic_like_ring, small_ring
from workloads.bunch import random_spins
from workloads.lattice import quad, sbend

pytestmark = pytest.mark.gpu

STRONG = [sbend(1.5, 0.45, 8, 4), quad(0.7, 9.0, "mk", 4, 3), sbend(2.0, 0.6, 8, 3, eta=1.1),
          quad(0.9, -9.0, "dkd", 8, 3)]       # elements with bounds that no lane meets


@pytest.mark.parametrize("ring,scale,aperture", [(rhic_like_ring(), 3.0, 0.05), (small_ring(), 6.0, 0.25),
                                                 (small_ring(quad_slices=4, rows=3, quad_method="mk"), 10.0, 9.0),
                                                 *(([e], 1.0, 9.0) for e in STRONG)])
def test_wide_bunches_match_the_oracle(ring, scale, aperture):
    beam = Beam(aperture=aperture)
    z, _, a = gaussian_bunch(1000, 19, beam, scale=scale)
    s = random_spins(1000, 20, math.pi)
    g = gpu_run(ring, beam, z, s, a, want_q=True)
    o = oracle.track(ring, beam, z, s, a, want_quaternion=True)
    assert_parity(g, o)
    live = o["alive"] == 1
    assert live.mean() > 0.3
    assert np.abs(g["q"] - o["q"])[:, live].max() <= 1e-10


def test_a_wide_bunch_takes_about_the_time_of_a_narrow_one():
    # 65536 particles, a wave per SIMD, no losses.  One body for all lanes of a wave
    # costs the rest of the series, two bodies twice the time.
    import torch
    from paper_1501_03450_amd import SpinTracker
    beam, n = Beam(aperture=3.0), 65536
    tr = SpinTracker(rhic_like_ring(sext_k2l=0.0), beam)
    best = {}
    for scale in (0.3, 4.0):
        z, s, a = gaussian_bunch(n, 5, beam, scale=scale)
        tr.set_particles(z, s, a)
        z0 = tr.z.clone()
        times = []
        for _ in range(6):
            tr.z.copy_(z0)
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            tr.track(1)
            e1.record()
            torch.cuda.synchronize()
            times.append(e0.elapsed_time(e1))
        assert (tr.alive == 1).all()
        best[scale] = min(times)
    tr.close()
    assert best[4.0] <= 1.6 * best[0.3], best
