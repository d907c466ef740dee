"""A lattice with every kind of extended element (drift-kick bends, piece-wise
constant spin, fourth-order quadrupoles, solenoids, rectangular bends, fringes) in
bunches small enough for the four-wave teams against the same particles in a bunch
that runs in blocks: the same bits.
"""

import math

import numpy as np
import pytest

from workloads import Beam, gaussian_bunch
from workloads.bunch import random_spins
from workloads.lattice import drift, quad, rbend, sbend, snake, solenoid, thin

pytestmark = pytest.mark.gpu

BIG = 32768 + 256            # more lanes than the teams take
TH = 2 * math.pi / 32
PARTS = [sbend(10.0, TH, 8, 3, method="teapot"), sbend(10.0, TH, 8, 1, method="teapot", spin="kick"),
         sbend(10.0, TH, 16, 1, method="teapot", spin="midpoint"), sbend(9.45, 0.0238, 8, 1, spin="midpoint"),
         quad(1.0, 0.05, "dkd", 8, 1, spin="kick"), quad(1.0, -0.05, "dkd", 4, 1, spin="midpoint"),
         quad(1.1, 0.08, "mk", 4, 1, spin="midpoint"), quad(1.1, -0.08, "mk", 6, 1, spin="midpoint"),
         solenoid(2.1, 0.016, 4, 2), rbend(3.0, 0.12, 8, 3), rbend(3.0, 0.12, 5, 1, spin="midpoint"),
         sbend(10.0, TH, 8, 3, fringe=True), quad(1.1, -0.08, "mk", 4, 2, fringe=True),
         quad(1.0, 0.05, "dkd4", 4, 2), quad(1.1, 0.05, "mk4", 4, 3), quad(1.1, -0.05, "mk4", 4, 3),
         sbend(10.0, TH, 8, 3), quad(1.0, 0.05, "dkd", 8, 3), thin(k2l=0.3), snake(math.pi, 0.3)]
RING = [e for part in PARTS for e in (part, drift(0.5))]


def run(beam, z, s, a, turns):
    import torch
    from paper_1501_03450_amd import SpinTracker
    tr = SpinTracker(RING, beam, report_every=2)
    tr.set_particles(z, s, a)
    q = tr.enable_quaternions()
    tr.track(turns)
    torch.cuda.synchronize()
    out = tr.read() + (q.cpu().numpy(),)
    tr.close()
    return out


@pytest.mark.parametrize("scale,aperture", [(1.0, 0.25), (6.0, 0.03)])
def test_extended_elements_have_the_same_bits_in_teams_and_blocks(scale, aperture):
    beam = Beam(aperture=aperture)
    z, _, a = gaussian_bunch(BIG, 31, beam, scale=scale)
    s = random_spins(BIG, 32, math.pi)
    a[5::97] = -7
    a[64:128] = 0
    big = run(beam, z, s, a, 3)
    for n in (1, 65, 1000):
        small = run(beam, z[:, :n], s[:, :n], a[:n], 3)
        for k in range(4):
            np.testing.assert_array_equal(small[k], big[k][..., :n], err_msg=f"n={n} output {k}")
