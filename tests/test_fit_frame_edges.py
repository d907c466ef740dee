"""The affine frame fit at the sizes where its kernels change path: fewer
samples than one wave's round, remainders of 4 and 32, one and many blocks, and
every input width.

Tolerance: the normal equations of standard normal inputs and targets of order
one have a condition below 1e3 at these sizes, so double-precision sums and the
solve leave below 1e-11; held to 1e-10.
"""

import numpy as np
import pytest

from oracle import mlp_ref as M

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_in", range(1, 9))
@pytest.mark.parametrize("extra", [0, 1, 3, 479, 4096, 70001])
def test_fit_matches_the_reference(n_in, extra):
    import torch
    from paper_1501_03450_amd import binding as B
    n = 8 * (n_in + 1) + extra
    rng = np.random.default_rng(100 * n_in + extra)
    x = rng.standard_normal((n, n_in)).astype(np.float32)
    t = (x @ rng.standard_normal((n_in, 4)) + 0.1 * rng.standard_normal((n, 4)) + 0.5).astype(np.float32)
    dx, dt = torch.as_tensor(x).cuda(), torch.as_tensor(t).cuda()
    m = B.st_mlp_create(0, n_in, 256, seed=1)
    f = B.st_mlp_fit_frame(m, dx.data_ptr(), dt.data_ptr(), n, 1e-5)
    B.st_mlp_destroy(m)
    r = M.fit_frame(x, t, 1e-5)
    for key in ("ref", "resid_rms", "resid_max", "scale"):
        np.testing.assert_allclose(np.array(f[key]), np.asarray(r[key]), rtol=0, atol=1e-10)
    np.testing.assert_allclose(np.array(f["lin"])[:, :n_in], np.asarray(r["lin"])[:, :n_in], rtol=0, atol=1e-10)
