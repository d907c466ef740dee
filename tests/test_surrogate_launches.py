"""Surrogate turns whose two kinds of lanes run beside each other in one launch
against the same particles in bunches that take two (more network lanes than the
shared launch takes, more fallback lanes than run in teams): a particle's turns do
not depend on the others, so every output has the same bits.
"""

import math

import numpy as np
import pytest

from workloads import Beam, gaussian_bunch, small_ring
from workloads.bunch import random_spins

pytestmark = pytest.mark.gpu

BESIDE, TEAM = 131072, 32768
N = BESIDE + TEAM + 4000


def run(z, s, a, fb, turns):
    import torch
    from paper_1501_03450_amd import SpinTracker
    from paper_1501_03450_amd import binding as B
    m = B.st_mlp_create(0, 6, 256, seed=3)
    tr = SpinTracker(small_ring(), Beam(aperture=0.03))
    tr.set_particles(z, s, a)
    d = torch.as_tensor(fb).cuda()
    inv = 1.0 / np.array([1e-3, 1e-4, 1e-3, 1e-4, 1e-2, 1e-3])
    B.st_track_surrogate(tr.ctx, m, turns, 1000, 1e9, np.zeros(6), inv, 0.0, d.data_ptr(),
                         torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    out = tr.read() + (d.cpu().numpy(),)
    tr.close()
    B.st_mlp_destroy(m)
    return out


@pytest.mark.parametrize("n_fallback", [300, TEAM + 300])
def test_lanes_beside_each_other_have_the_bits_of_separate_launches(n_fallback):
    z, _, a = gaussian_bunch(N, 71, Beam(aperture=0.03), scale=3.0)    # some are lost on the way
    s = random_spins(N, 72, math.pi)
    a[5::997] = -3
    fb = np.zeros(N, dtype=np.int32)
    fb[:n_fallback] = -1
    big = run(z, s, a, fb, 6)
    assert (big[2] < 0).sum() > (a < 0).sum()
    for lo, hi in ((0, 300), (200, 1500), (n_fallback - 64, n_fallback + 65), (n_fallback - 1, n_fallback + 3)):
        part = run(z[:, lo:hi], s[:, lo:hi], a[lo:hi], fb[lo:hi], 6)
        for k in range(4):
            np.testing.assert_array_equal(part[k], big[k][..., lo:hi], err_msg=f"{lo}..{hi} output {k}")
