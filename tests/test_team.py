"""Bunches small enough for the four-wave teams against the same particles
inside a bunch that runs in blocks: the same bits in orbit, spin, status and
one-turn quaternion, on rings that reach every path of the element loop.
"""

import math

import numpy as np
import pytest

from workloads import Beam, gaussian_bunch, rhic_like_ring, small_ring
from workloads.bunch import random_spins
from workloads.lattice import Element, drift, quad, sbend, snake, thin

pytestmark = pytest.mark.gpu

BIG = 32768 + 256            # more lanes than the teams take
LOSSY = small_ring()[:8] + [thin(k2l=3.0)] + small_ring()[8:40] + [thin(k2l=-3.0)] + small_ring()[40:]
RINGS = {
    "rhic": (rhic_like_ring(), 2, 1.0, 0.05),
    "small": (small_ring(), 7, 1.0, 0.05),
    "lossy": (LOSSY, 9, 3.0, 0.03),                       # losses in many elements and turns
    "general": (small_ring(quad_slices=6, bend_slices=4, rows=3, quad_method="mk"), 3, 2.0, 0.05),
    "mixed_lanes": ([quad(1.1, 0.25, "mk", 4, 3), drift(1.0), sbend(9.45, 0.0238, 8, 4), drift(2.0),
                     quad(1.1, -0.25, "mk", 4, 3), drift(0.0)] * 9, 3, 6.0, 0.3),
    "drifts": ([drift(1.0)] * 150 + [snake(math.pi, 0.3)] + [drift(0.5), Element("marker")] * 70, 3, 1.0, 0.05),
    "thin_run": ([thin(k1l=0.01), thin(k2l=0.3)] * 40 + [Element("marker")], 2, 1.0, 0.05),
    "one_element": ([sbend(9.45, 0.0238, 8, 4)], 5, 1.0, 0.05),
    "only_drift": ([drift(3.0)], 4, 20.0, 0.05),
}


def run(ring, beam, z, s, a, turns):
    import torch
    from paper_1501_03450_amd import SpinTracker
    tr = SpinTracker(ring, beam, report_every=2)
    tr.set_particles(z, s, a)
    q = tr.enable_quaternions()
    tr.track(turns)
    torch.cuda.synchronize()
    out = tr.read() + (q.cpu().numpy(), tr.polarization().cpu().numpy())
    tr.close()
    return out


@pytest.mark.parametrize("name", list(RINGS))
def test_a_small_bunch_has_the_bits_of_the_same_particles_in_a_large_one(name):
    ring, turns, scale, aperture = RINGS[name]
    beam = Beam(aperture=aperture)
    z, _, a = gaussian_bunch(BIG, 31, beam, scale=scale)
    s = random_spins(BIG, 32, math.pi)
    a[5::97] = -7                                          # lost before the call
    a[64:128] = 0                                          # a whole team
    big = run(ring, beam, z, s, a, turns)
    for n in (1, 63, 65, 1000):
        small = run(ring, beam, z[:, :n], s[:, :n], a[:n], turns)
        for k in range(4):
            np.testing.assert_array_equal(small[k], big[k][..., :n], err_msg=f"{name} n={n} output {k}")
        live = small[2] == 1
        if turns % 2 == 0 and live.any():
            np.testing.assert_allclose(small[4][-1, :3], small[1][:, live].mean(axis=1), rtol=0, atol=1e-13)
            assert small[4][-1, 3] == live.sum()
