"""Gradients that one sample dominates: the others' targets are the network's own
outputs, so that a tile that is left out, or taken twice, shows whole.  The sample
lies in the first and the last tile of a workgroup's rounds and in remainders.
"""

import numpy as np
import pytest

from oracle import mlp_ref as M
from test_train_tiles import Net, _rel, _samples

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,at", [(33, 32), (8193, 8192), (8193, 8191), (8224, 8193), (131073, 131072),
                                  (131073, 131071), (131072, 16384), (131104, 0)])
def test_the_gradient_has_every_tile_once(n, at):
    import torch
    net = Net(6, 61)
    x, t = _samples(n, 6, 8)
    dx, q = torch.as_tensor(x).cuda(), torch.empty((n, 4), dtype=torch.float32, device="cuda")
    net.B.st_mlp_infer(net.net, dx.data_ptr(), q.data_ptr(), n)
    torch.cuda.synchronize()
    t = q.cpu().numpy()
    t[at] = -t[at]                       # the farthest a target can be
    t[at] = np.roll(t[at], 1)            # (the very opposite has no gradient)
    whole = net.gradient(x, t)[0].astype(np.float64) * n
    one = net.gradient(x[at:at + 1], t[at:at + 1])[0].astype(np.float64)
    # the others' residuals are rounding, 1e-7 of this one's; over 131072 of them
    # they stay below 1e-2 of it even if they all add up
    for k, (a, b) in enumerate(zip(M.unflatten(whole, 6), M.unflatten(one, 6))):
        assert _rel(a, b) <= 2e-2, (k, _rel(a, b))
    net.B.st_mlp_destroy(net.net)
