"""Rounding errors of the slice loops that must not add up: a factor that is the
same in every slice (1/P, its products with an element's constants) acts, once
rounded, like an error of the particle's momentum, and the orbit, the flight time
or the spin drifts away in proportion to the path.  RMS over the bunch against the
extended-precision oracle, bounded by what a quarter of an ulp (2^-54) of such a
factor leads to.
"""

import math

import numpy as np
import pytest

import oracle
from test_parity_fp64 import gpu_run
from workloads import Beam, gaussian_bunch, rhic_like_ring, uniform_bend_ring
from workloads.bunch import random_spins
from workloads.lattice import sbend

pytestmark = pytest.mark.gpu

BEAM = Beam(aperture=2.0)
QUARTER_ULP = 2.0 ** -54


def errors(ring, turns, n=2048, only_energy=False):
    z, _, _ = gaussian_bunch(n, 7, BEAM)
    if only_energy:
        z[:5] = 0.0
    s = random_spins(n, 8, math.pi)
    g = gpu_run(ring, BEAM, z, s, turns=turns)
    o = oracle.track(ring, BEAM, z, s, turns=turns)
    np.testing.assert_array_equal(g["alive"], o["alive"])
    rms = np.sqrt(np.mean((g["z"] - o["z"]) ** 2, axis=1))
    return rms, np.sqrt(np.mean((g["spin"] - o["spin"]) ** 2))


@pytest.mark.parametrize("spin,rows", [("kick", 1), ("midpoint", 1), ("edges", 3)])
def test_drift_kick_bends_keep_the_momentum(spin, rows):
    # half a turn in 16 bends of radius rho: a momentum error d moves X by
    # 2 rho d and T by pi rho d
    th = 2.0 * math.pi / 32.0
    rms, _ = errors([sbend(10.0, th, 8, rows, method="teapot", spin=spin)] * 16, 1)
    rho = 10.0 / th
    assert rms[0] <= 2.0 * rho * QUARTER_ULP, rms[0]
    assert rms[4] <= math.pi * rho * QUARTER_ULP, rms[4]


@pytest.mark.parametrize("ring,turns", [(uniform_bend_ring(), 4), ([sbend(9.45, 0.0238, 8, 4)] * 64, 2),
                                        ([sbend(3.1, 0.077, 8, 3, eta=1.0003)] * 20, 2)])
def test_bends_turn_the_spin_by_the_whole_angle(ring, turns):
    # a factor off by d turns the spin by (1 + G gamma) times the bends' angle times
    # d too far
    _, spin = errors(ring, turns)
    angle = turns * sum(e.angle for e in ring)
    assert spin <= (1.0 + BEAM.G * BEAM.gamma0) * angle * QUARTER_ULP, spin


def test_flight_time_of_the_rhic_scale_ring_off_momentum():
    # Px changes by the momentum deviation times the angle in every bend, and T by
    # rho times that: 2.5 m a turn for one sigma, on which a common factor's
    # roundings act.  1.6 half ulps are two of them and the orbit's own noise
    # (half of it); the square of a rounded factor is above.
    rms, _ = errors(rhic_like_ring(), 2, only_energy=True)
    rho = 9.45 / (2.0 * math.pi / 264.0)
    assert rms[4] <= 1.6 * 2.0 ** -53 * 2 * 2.0 * math.pi * rho * 1e-3, rms[4]


def test_bends_at_the_edge_of_the_series_turn_the_spin_by_the_whole_angle():
    # the same bound where Px is close to the short series' limit of 3.6 mrad: a
    # series that stops a term early is off by 3e-16 of the angle there
    ring, beam, n = [sbend(2.0, -0.05, 8, 4)], Beam(gamma0=250.0, aperture=2.0), 2000
    rng = np.random.default_rng(5)
    z = np.zeros((6, n))
    z[1] = rng.choice([-1.0, 1.0], n) * rng.uniform(0.0032, 0.0035, n)
    s = random_spins(n, 3, math.pi)
    g, o = gpu_run(ring, beam, z, s), oracle.track(ring, beam, z, s)
    spin = np.sqrt(np.mean((g["spin"] - o["spin"]) ** 2))
    assert spin <= (1.0 + beam.G * beam.gamma0) * 0.05 * QUARTER_ULP, spin
