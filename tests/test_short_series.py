"""The short-series bodies of sector bends and quadrupoles at the edges of the
lanes they take: momenta, offsets and energies on both sides of every bound,
against the extended-precision oracle.

Tolerance: the method's own (test_parity_fp64), orbit 1e-12 · max(|z|, bunch
RMS) and spin components 1e-10 after one passage.
"""

import numpy as np
import pytest

import oracle
from test_parity_fp64 import assert_parity, gpu_run
from workloads import Beam
from workloads.bunch import random_spins
from workloads.lattice import quad, sbend

pytestmark = pytest.mark.gpu

ELEMENTS = {
    "bend_8x4": sbend(9.45, 0.0238, 8, 4), "bend_8x3": sbend(10.0, 0.196, 8, 3),
    "bend_reverse": sbend(2.0, -0.05, 8, 4), "bend_eta": sbend(9.45, 0.0238, 8, 4, eta=1.002),
    "mk_focus": quad(1.1, 0.08, "mk", 4, 4), "mk_defocus": quad(1.1, -0.08, "mk", 4, 3),
    "mk_strong": quad(0.5, 3.0, "mk", 4, 3),
    "dkd_focus": quad(1.0, 0.05, "dkd", 8, 3), "dkd_defocus": quad(1.0, -0.05, "dkd", 8, 3),
    "dkd_strong": quad(0.5, -3.0, "dkd", 8, 3),
}
BEAMS = {"proton": Beam(aperture=2.0), "slow": Beam(gamma0=1.3, aperture=2.0),
         "deuteron": Beam(G=-0.143, gamma0=12.0, aperture=2.0),
         "fast": Beam(gamma0=250.0, aperture=2.0)}


def edge_bunch(beam, n=3072, seed=11):
    rng = np.random.default_rng(seed)
    sign = lambda: rng.choice([-1.0, 1.0], n)                       # noqa: E731
    mom = [0.0, 1e-9, 1e-5, 3e-4, 0.0034, 0.0035999, 0.0036001, 0.0066, 0.0071, 0.0073, 0.0156]
    pos = [0.0, 1e-9, 1e-4, 3e-3, 0.01, 0.03, 0.05, 0.0535, 0.2]
    c3 = sign() * rng.choice([0.0, 1e-9, 2e-3, 8e-3, 0.1249999, 0.1250001, 0.3], n)
    z = np.empty((6, n))
    z[0], z[2] = sign() * rng.choice(pos, n), sign() * rng.choice(pos, n)
    z[1], z[3] = sign() * rng.choice(mom, n), sign() * rng.choice(mom, n)
    z[4] = 1e-2 * rng.standard_normal(n)
    ib = 1.0 / beam.beta0
    z[5] = c3 / (ib + np.sqrt(ib * ib + c3))                        # P² - 1 = c3
    return z


# (not the strong quadrupoles at gamma 250: a slice there turns the spin of the
# outermost lanes by tens of radians, beyond what the general body's argument
# halving keeps to 1e-10)
@pytest.mark.parametrize("name,beam_name", [(e, b) for e in ELEMENTS for b in BEAMS
                                            if not (e.endswith("strong") and b == "fast")])
def test_both_sides_of_every_bound_match_the_oracle(name, beam_name):
    beam, ring = BEAMS[beam_name], [ELEMENTS[name]]
    z = edge_bunch(beam)
    s = random_spins(z.shape[1], 3, np.pi)
    g = gpu_run(ring, beam, z, s)
    o = oracle.track(ring, beam, z, s)
    assert_parity(g, o, f"{name} {beam_name}")
    # a lane's result does not depend on the body its neighbours take
    order = np.random.default_rng(5).permutation(z.shape[1])[:1000]
    h = gpu_run(ring, beam, z[:, order], s[:, order])
    np.testing.assert_array_equal(h["z"], g["z"][:, order])
    np.testing.assert_array_equal(h["spin"], g["spin"][:, order])
