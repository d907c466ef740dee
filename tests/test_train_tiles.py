"""Gradients at the edges of the training kernels' tiles: remainders of the 16
rows of a matrix instruction and of the 32-sample tile, numbers of inputs that
fill the padded eight or leave one, one tile per workgroup and one more, and the
size from which there is a second round of workgroups.
"""

import numpy as np
import pytest

from oracle import mlp_ref as M

pytestmark = pytest.mark.gpu


def _samples(n, n_in, seed):
    """Targets about one direction: the gradient is a coherent sum."""
    rng = np.random.default_rng(seed)
    x = (1.0 + 0.3 * rng.normal(size=(n, n_in))).astype(np.float32)
    t = np.array([1.0, 2.0, 3.0, 4.0]) + 0.2 * rng.normal(size=(n, 4))
    return x, (t / np.linalg.norm(t, axis=1, keepdims=True)).astype(np.float32)


class Net:
    def __init__(self, n_in, seed):
        from paper_1501_03450_amd import binding as B
        self.B, self.n_in = B, n_in
        self.net = B.st_mlp_create(0, n_in, 256, seed=seed)
        self.theta = np.empty(B.st_mlp_params(self.net), dtype=np.float32)
        B.st_mlp_params(self.net, self.theta.ctypes.data, None)

    def gradient(self, x, t):
        import torch
        g = torch.zeros(self.theta.size, dtype=torch.float32, device="cuda")
        loss = torch.zeros(1, dtype=torch.float32, device="cuda")
        dx, dt = torch.as_tensor(x).cuda(), torch.as_tensor(t).cuda()
        self.B.st_mlp_gradient(self.net, dx.data_ptr(), dt.data_ptr(), len(x), g.data_ptr(), loss.data_ptr())
        torch.cuda.synchronize()
        return g.cpu().numpy(), loss.item()


def _rel(a, b):
    return np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-30)


@pytest.mark.parametrize("n_in", [1, 6, 8])
def test_gradient_of_ragged_batches_matches_the_cpu_reference(n_in):
    # the repository's tolerance of a gradient against this reference, tensor by
    # tensor: 1e-2 (bf16 rounding that falls on the other side)
    net = Net(n_in, 50 + n_in)
    p = M.unflatten(net.theta.astype(np.float64), n_in)
    p[2], p[4] = M.bf16_round(p[2]), M.bf16_round(p[4])
    for n in (1000, 33, 64, 31, 97, 500):        # the scratch of a larger batch serves the smaller
        x, t = _samples(n, n_in, n)
        g, loss = net.gradient(x, t)
        x, t = x.astype(np.float64), t.astype(np.float64)
        ref = M.backward(p, x, t, None, None, round_act=M.bf16_round, round_dz=M.bf16_round,
                         round_ds=M.bf16_round)
        for k, (a, b) in enumerate(zip(M.unflatten(g, n_in), ref)):
            assert _rel(a, b) <= 1e-2, (n, k, _rel(a, b))
        want = M.loss(p, x, t, None, None, round_act=M.bf16_round)
        assert abs(loss - want) <= 1e-3 * max(1.0, want)
    net.B.st_mlp_destroy(net.net)


@pytest.mark.parametrize("n,h", [(8192, 4096), (8193, 8192), (131072, 65536), (131073, 1000)])
def test_gradient_across_the_workgroup_rounds_is_the_weighted_mean_of_its_parts(n, h):
    # the mean loss is linear in the per-sample terms, whose rounding does not
    # depend on the batch; what differs is the order of fp32 sums (1e-4, as for
    # larger batches)
    net = Net(6, 60)
    x, t = _samples(n, 6, 7)
    whole = net.gradient(x, t)[0].astype(np.float64)
    parts = (h * net.gradient(x[:h], t[:h])[0].astype(np.float64) +
             (n - h) * net.gradient(x[h:], t[h:])[0].astype(np.float64)) / n
    for k, (a, b) in enumerate(zip(M.unflatten(whole, 6), M.unflatten(parts, 6))):
        assert _rel(a, b) <= 1e-4, (k, _rel(a, b))
    net.B.st_mlp_destroy(net.net)
