"""Network inference at the edges of its tiles: one sample, remainders of the 16
rows of a matrix instruction and of the 32- and 64-sample tiles, more tiles than
workgroups, and both sides of the rule that picks the tile.  A sample's result
does not depend on the batch around it (its own column of every product), so each
batch has to give the bits of the same samples in another batch; one of them is
held to the CPU reference.
"""

import numpy as np
import pytest

from oracle import mlp_ref as M

pytestmark = pytest.mark.gpu

SIZES = (1, 15, 17, 32, 33, 63, 65, 8191, 8193, 16385, 24576, 24577, 32767, 49153, 70001)


@pytest.mark.parametrize("n_in", [1, 4, 6, 8])
def test_a_sample_has_the_same_bits_in_batches_of_any_size(n_in):
    import torch
    from paper_1501_03450_amd import binding as B
    m = B.st_mlp_create(0, n_in, 256, seed=40 + n_in)
    theta = np.empty(M.n_params(n_in), dtype=np.float32)
    B.st_mlp_params(m, theta.ctypes.data, None)
    theta[-4:] = (0.5, -0.5, 0.5, 0.5)       # outputs of unit size, as a trained network has
    B.st_mlp_params(m, None, theta.ctypes.data)
    x = np.random.default_rng(5).standard_normal((max(SIZES), n_in)).astype(np.float32)
    dx = torch.as_tensor(x).cuda()

    def infer(n):
        q = torch.full((n + 64, 4), -7.0, dtype=torch.float32, device="cuda")
        B.st_mlp_infer(m, dx.data_ptr(), q.data_ptr(), n)
        torch.cuda.synchronize()
        assert (q[n:] == -7.0).all(), f"n={n}: written past the end"
        return q[:n].cpu().numpy()

    whole = infer(max(SIZES))
    for n in SIZES:
        np.testing.assert_array_equal(infer(n), whole[:n], err_msg=f"n={n}")
    p = M.unflatten(theta.astype(np.float64), n_in)
    p[2], p[4] = M.bf16_round(p[2]), M.bf16_round(p[4])      # as the kernels use them
    q, _ = M.forward(p, x[:2000].astype(np.float64), round_act=M.bf16_round)
    assert np.abs(whole[:2000] - q).max() < 1e-3
    B.st_mlp_destroy(m)
