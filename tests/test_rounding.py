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
from workloads import Beam, gaussian_bunch
from workloads.bunch import random_spins
from workloads.lattice import sbend

pytestmark = pytest.mark.gpu

BEAM = Beam(aperture=2.0)
QUARTER_ULP = 2.0 ** -54


def errors(ring, turns, n=2048):
    z, _, _ = gaussian_bunch(n, 7, BEAM)
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
