"""Surrogate turns and replays on both sides of the number of lanes up to which
they run in four-wave teams (8192 in surrogate tracking), against the same particles
in small bunches: a particle's turns do not depend on the others, so every output
has the same bits.
"""

import math

import numpy as np
import pytest

from workloads import Beam, gaussian_bunch, small_ring
from workloads.bunch import random_spins

pytestmark = pytest.mark.gpu

TEAM = 8192
BEAM = Beam(aperture=0.03)


def run(z, s, a, fb, turns, audit, threshold):
    import torch
    from paper_1501_03450_amd import SpinTracker
    from paper_1501_03450_amd import binding as B
    m = B.st_mlp_create(0, 6, 256, seed=3)
    tr = SpinTracker(small_ring(), BEAM)
    tr.set_particles(z, s, a)
    d = torch.as_tensor(fb).cuda()
    inv = 1.0 / np.array([1e-3, 1e-4, 1e-3, 1e-4, 1e-2, 1e-3])
    B.st_track_surrogate(tr.ctx, m, turns, audit, threshold, np.zeros(6), inv, 0.0, d.data_ptr(),
                         torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    out = tr.read() + (d.cpu().numpy(),)
    tr.close()
    B.st_mlp_destroy(m)
    return out


def compare(n, n_fallback, audit, threshold):
    z, s, a = gaussian_bunch(n, 73, BEAM, scale=2.0)
    s = random_spins(n, 74, math.pi)
    fb = np.zeros(n, dtype=np.int32)
    fb[:n_fallback] = -1
    whole = run(z, s, a, fb, 5, audit, threshold)
    for lo, hi in ((0, 200), (TEAM - 100, min(n, TEAM + 60))):
        part = run(z[:, lo:hi], s[:, lo:hi], a[lo:hi], fb[lo:hi], 5, audit, threshold)
        for k in range(4):
            np.testing.assert_array_equal(part[k], whole[k][..., lo:hi], err_msg=f"{lo}..{hi} output {k}")


@pytest.mark.parametrize("n_fallback", [TEAM, TEAM + 1])
def test_fallback_lanes_beside_network_lanes(n_fallback):
    compare(n_fallback + 3000, n_fallback, 1000, 1e9)


@pytest.mark.parametrize("n", [TEAM, TEAM + 1])
def test_audits_and_replays(n):
    compare(n, 0, 2, 0.0)                # every particle fails every audit
