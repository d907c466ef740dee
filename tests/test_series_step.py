"""Slices of the general and the extended bodies with lanes on both sides of the
bounds of their short series (transverse momenta about 2^-6 and 2^-4.5 of P, bend
angles about 0.03 rad a step), against the extended-precision oracle.

Tolerance: the method's own (test_parity_fp64), orbit 1e-12 · max(|z|, bunch RMS)
and spin components 1e-10 after one passage.
"""

import numpy as np
import pytest

import oracle
from test_parity_fp64 import assert_parity, gpu_run
from workloads import Beam
from workloads.bunch import random_spins
from workloads.lattice import drift, quad, sbend, solenoid

pytestmark = pytest.mark.gpu

BEAM = Beam(aperture=5.0)
TH = 0.196
ELEMENTS = {
    "drift": drift(2.0),
    "teapot_kick": sbend(10.0, TH, 8, 1, method="teapot", spin="kick"),
    "teapot_kick_4": sbend(10.0, TH, 4, 1, method="teapot", spin="kick"),
    "teapot_midpoint": sbend(10.0, TH, 5, 1, method="teapot", spin="midpoint"),
    "teapot_edges": sbend(10.0, TH, 8, 3, method="teapot"),
    "teapot_closed": sbend(10.0, TH, 2, 1, method="teapot", spin="kick"),
    "teapot_closed_edges": sbend(2.0, 0.9, 1, 1, method="teapot"),
    "dkd_kick": quad(1.0, 0.05, "dkd", 4, 1, spin="kick"),
    "dkd_midpoint": quad(1.0, -0.05, "dkd", 3, 1, spin="midpoint"),
    "dkd_edges": quad(1.0, 0.05, "dkd", 6, 2),
    "dkd4_edges": quad(1.0, 0.05, "dkd4", 4, 2),
    "mk_midpoint": quad(1.1, 0.08, "mk", 3, 1, spin="midpoint"),
    "mk_edges": quad(1.1, -0.08, "mk", 6, 2),
    "mk4_midpoint": quad(1.1, -0.08, "mk4", 2, 1, spin="midpoint"),
    "bend_midpoint": sbend(5.0, 0.3, 4, 1, spin="midpoint"),
    "bend_edges": sbend(5.0, 0.3, 6, 2),
    "solenoid": solenoid(2.1, 0.016, 4, 2),
}


def edge_bunch(n=3072, seed=13):
    rng = np.random.default_rng(seed)
    sign = lambda: rng.choice([-1.0, 1.0], n)                       # noqa: E731
    mom = [0.0, 1e-5, 3e-4, 0.0033, 0.0155, 0.015625, 0.0158, 0.0195, 0.0315, 0.044, 0.0443, 0.2]
    z = np.empty((6, n))
    z[0], z[2] = sign() * rng.choice([0.0, 1e-4, 0.01, 0.1], n), sign() * rng.choice([0.0, 1e-4, 0.01, 0.1], n)
    z[1], z[3] = sign() * rng.choice(mom, n), sign() * rng.choice(mom[:8], n)
    z[4] = 1e-2 * rng.standard_normal(n)
    c3 = sign() * rng.choice([0.0, 1e-9, 2e-3, 0.1], n)
    ib = 1.0 / BEAM.beta0
    z[5] = c3 / (ib + np.sqrt(ib * ib + c3))                        # P² - 1 = c3
    return z


@pytest.mark.parametrize("name", list(ELEMENTS))
def test_lanes_about_the_series_bounds_match_the_oracle(name):
    ring, z = [ELEMENTS[name]], edge_bunch()
    s = random_spins(z.shape[1], 3, np.pi)
    g = gpu_run(ring, BEAM, z, s)
    o = oracle.track(ring, BEAM, z, s)
    assert_parity(g, o, name)
    # a lane's result does not depend on what its neighbours need
    order = np.random.default_rng(5).permutation(z.shape[1])[:1000]
    h = gpu_run(ring, BEAM, z[:, order], s[:, order])
    np.testing.assert_array_equal(h["z"], g["z"][:, order])
    np.testing.assert_array_equal(h["spin"], g["spin"][:, order])
    alone = gpu_run(ring, BEAM, z[:, 5:6], s[:, 5:6])
    np.testing.assert_array_equal(alone["z"], g["z"][:, 5:6])
    np.testing.assert_array_equal(alone["spin"], g["spin"][:, 5:6])
