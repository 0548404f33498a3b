"""The layer products (forward, backward, update) at the edges of their tiles.

Networks without preconditioners: the gradient of the last layer is O^T X (update product behind one forward product
per layer), that of the first layer also contains the backward product.  Compared with the float64 oracle.
"""
import numpy as np
import pytest

import workloads
from oracle.network import NGSGDNetwork

pytestmark = pytest.mark.gpu

# Every product forms its sums with a relative error of at most 2.5e-7 of the result's norm; a gradient is behind at most
# four of them (forward, forward, backward, update) and two element-wise functions accurate to a few 2^-24.
TOL = 2e-6

# (minibatch, input, hidden, classes): below, at and above the tile sizes 32, 64, 96, 128 and the K-blocks of 32 and 64;
# then shapes whose tile counts select the larger tiles
SHAPES = [(1, 4, 3, 2), (2, 8, 33, 5), (31, 36, 33, 17), (32, 64, 32, 64), (33, 60, 65, 31), (63, 64, 95, 97), (65, 68, 127, 129),
          (96, 128, 191, 193), (129, 256, 257, 63), (200, 300, 1000, 259), (512, 360, 3001, 1009), (515, 1024, 2051, 333),
          (1027, 700, 2050, 301), (300, 2048, 2040, 300)]


def rel(a, b):
    return float(np.linalg.norm(a.astype(np.float64) - b) / np.linalg.norm(b))


@pytest.mark.parametrize("n,din,hidden,classes", SHAPES)
def test_gradients_of_a_plain_network(ngsgd, n, din, hidden, classes):
    import torch
    rng = np.random.default_rng(n * 7 + hidden)
    dims = [din, hidden, classes]
    weights = [rng.standard_normal((dims[l + 1], dims[l] + 1)).astype(np.float32) / np.float32(np.sqrt(dims[l] + 1)) for l in range(2)]
    x = rng.standard_normal((n, din)).astype(np.float32)
    y = rng.integers(0, classes, n).astype(np.int32)
    ora = NGSGDNetwork(dims, [workloads.TANH], weights, rank_in=0, rank_out=0)
    gpu = ngsgd.Network(dims, [ngsgd.NGSGD_TANH], n, rank_in=0, rank_out=0)
    for l, w in enumerate(weights):
        gpu.set_params(l, torch.from_numpy(w).cuda())
    obj = ora.step(x, y, 0.01)
    out = gpu.step(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), 0.01)
    torch.cuda.synchronize()
    assert abs(float(out.item()) - obj) < 2e-6 * abs(obj) + 1e-6
    for l in range(2):
        assert rel(gpu.last_gradient(l).cpu().numpy(), ora.last["delta"][l]) < TOL, l
        assert rel(gpu.get_params(l).cpu().numpy(), ora.W[l]) < TOL, l
