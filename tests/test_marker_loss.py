"""The loss check of a marker, which leads the lattice: particles that start
outside the aperture or with a non-finite coordinate are lost in element 0 and keep
their state, also those that the drift behind it would bring back inside.

In teams (1000 particles) and blocks (33024), in double and mixed precision, in an
extended lattice, and in surrogate tracking on and off the network, against the
oracle.  Orbit 1e-12 · max(|z|, bunch RMS) and spin 1e-10 after one turn.
"""

import math

import numpy as np
import pytest

import oracle
from test_parity_fp64 import assert_parity
from workloads import Beam, gaussian_bunch, small_ring
from workloads.bunch import random_spins
from workloads.lattice import Element, drift, quad, sbend

pytestmark = pytest.mark.gpu

MARKER = Element("marker")
BEAM = Beam(aperture=0.05)
RINGS = {
    "before_drift": [MARKER, drift(1.0)],
    "alone": [MARKER],
    "two": [MARKER, MARKER, drift(1.0), MARKER],
    "before_bend": [MARKER, sbend(9.45, 0.0238, 8, 4), drift(0.5)],
    "before_ring": [MARKER] + small_ring()[:24] + [MARKER, MARKER] + small_ring()[24:48],
    "extended": [MARKER, drift(1.0), quad(1.0, 0.05, "dkd", 4, 1, spin="kick"), MARKER, drift(1.0)],
}


def bunch(n):
    z, _, a = gaussian_bunch(n, 41, BEAM)
    z[0, 0::13], z[1, 0::13] = 0.06, -0.02           # back inside after 1 m
    z[2, 1::13], z[3, 1::13] = -0.06, 0.02
    z[0, 2::13] = 0.06
    z[0, 3::13] = 0.049
    a[4::13] = -5
    z[0, 5::97], z[1, 6::97], z[2, 7::97] = np.nan, np.inf, -np.inf
    z[3, 8::97], z[4, 9::97], z[4, 10::97] = np.nan, np.nan, np.inf
    return z, random_spins(n, 42, math.pi), a


def tracker(ring, z, s, a, precision="fp64"):
    from paper_1501_03450_amd import SpinTracker
    tr = SpinTracker(ring, BEAM, precision=precision)
    tr.set_particles(z, s, a)
    return tr


def check(got, z, s, a, ref, spin_tol=True):
    zg, sg, ag = got
    np.testing.assert_array_equal(ag, ref["alive"])
    out = (a == 1) & (ag == -1)                      # lost in the marker: as they came
    assert out.sum() > len(a) / 8
    np.testing.assert_array_equal(zg[:, out], z[:, out])
    np.testing.assert_array_equal(sg[:, out], s[:, out])
    live = ag == 1
    assert live.sum() > len(a) / 3
    assert_parity(dict(z=zg[:, live], spin=sg[:, live] if spin_tol else ref["spin"][:, live], alive=ag[live]),
                  dict(z=ref["z"][:, live], spin=ref["spin"][:, live], alive=ref["alive"][live]))


@pytest.mark.parametrize("precision", ["fp64", "mixed_all"])
@pytest.mark.parametrize("n", [1000, 33024])
@pytest.mark.parametrize("name", list(RINGS))
def test_a_leading_marker_loses_what_starts_outside(name, n, precision):
    import torch
    z, s, a = bunch(n)
    tr = tracker(RINGS[name], z, s, a, precision)
    q = tr.enable_quaternions()
    tr.track(1)
    torch.cuda.synchronize()
    got, q = tr.read(), q.cpu().numpy()
    tr.close()
    ref = oracle.track(RINGS[name], BEAM, z, s, a, want_quaternion=True)
    check(got, z, s, a, ref, precision == "fp64")
    out = (a == 1) & (got[2] == -1)
    np.testing.assert_array_equal(q[:, out], np.array([[1.0], [0.0], [0.0], [0.0]]) * np.ones(out.sum()))


@pytest.mark.parametrize("n", [1000, 33024])
@pytest.mark.parametrize("name", ["before_drift", "alone", "before_ring", "extended"])
def test_a_leading_marker_in_surrogate_tracking(name, n):
    import torch
    from paper_1501_03450_amd import binding as B
    z, s, a = bunch(n)
    m = B.st_mlp_create(0, 6, 256, seed=3)
    for audit, start in ((1, 0), (1000, 0), (1000, 1)):
        # audited in every turn against a threshold that no network meets; on the
        # network between the first and the last turn; every particle falling back
        tr = tracker(RINGS[name], z, s, a)
        fb = torch.full((n,), start, dtype=torch.int32, device="cuda")
        inv = 1.0 / np.array([1e-3, 1e-4, 1e-3, 1e-4, 1e-2, 1e-3])
        B.st_track_surrogate(tr.ctx, m, 4, audit, 0.0 if audit == 1 else 1e9, np.zeros(6), inv, 0.0,
                             fb.data_ptr(), torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        got = tr.read()
        tr.close()
        ref = oracle.track(RINGS[name], BEAM, z, s, a, turns=4)
        np.testing.assert_array_equal(got[2], ref["alive"])
        out = (a == 1) & (got[2] == -1)
        np.testing.assert_array_equal(got[0][:, out], z[:, out])
        np.testing.assert_array_equal(got[1][:, out], s[:, out])
    B.st_mlp_destroy(m)
