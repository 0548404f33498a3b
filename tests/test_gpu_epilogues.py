"""GPU parity of what the products and the finishing kernel do beside their sums: tanh and its derivative, the maximum change of a
layer (App. C.3), the scaling by gamma of rows of any length.  Against the float64 oracle.
"""
import numpy as np
import pytest

import workloads
from oracle.network import NGSGDNetwork
from oracle.online_ng import OnlineNaturalGradient
from test_gpu_fused_apply import data, gpu_call
from test_gpu_layer_products import TOL, plain_pair, rel

pytestmark = pytest.mark.gpu

# (minibatch, hidden, classes): the backward product with the derivative in its epilogue on each of its tiles, then in K splits with
# the derivative behind them
BACKWARD = [(7, 4, 42), (388, 1276, 20), (386, 2440, 21), (585, 2474, 67), (972, 2110, 65),
            (8, 4, 346), (1074, 5, 418), (2, 2120, 387), (65, 1778, 580)]


def random_weights(rng, dims):
    return [rng.standard_normal((dims[l + 1], dims[l] + 1)).astype(np.float32) / np.float32(np.sqrt(dims[l] + 1)) for l in range(len(dims) - 1)]


def both_gradients(ora, gpu, x, y):
    import torch
    ora.step(x, y, 0.01)
    gpu.step(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), 0.01)
    return ora.last["delta"], [gpu.last_gradient(l).cpu().numpy() for l in range(2)]


@pytest.mark.parametrize("n,hidden,classes", BACKWARD)
def test_derivative_of_tanh(ngsgd, n, hidden, classes):
    rng = np.random.default_rng(9000 + n + hidden)
    dims = [20, hidden, classes]
    ora, gpu = plain_pair(ngsgd, dims, random_weights(rng, dims), n)
    x = rng.standard_normal((n, dims[0])).astype(np.float32)
    y = rng.integers(0, classes, n).astype(np.int32)
    want, got = both_gradients(ora, gpu, x, y)
    for l in range(2):
        assert rel(got[l], want[l]) < TOL, l


@pytest.mark.parametrize("n,din,hidden,classes", [(1, 4, 3, 2), (33, 60, 65, 31), (65, 68, 127, 129), (200, 300, 1000, 259), (515, 400, 2051, 333)])
def test_maximum_change(ngsgd, n, din, hidden, classes):
    """The sum of |o_i| |x_i| over the rows is of positive terms, each from two sums of squares: 1e-6 covers both."""
    import torch
    rng = np.random.default_rng(9500 + n + hidden)
    dims = [din, hidden, classes]
    weights = random_weights(rng, dims)
    for limit in (1.0e-3, 1.0e3):   # all layers scaled, none
        ora = NGSGDNetwork(dims, [workloads.TANH], weights, rank_in=0, rank_out=0, max_change_per_sample=limit)
        gpu = ngsgd.Network(dims, [workloads.TANH], n, rank_in=0, rank_out=0, max_change_per_sample=limit)
        for l, w in enumerate(weights):
            gpu.set_params(l, torch.from_numpy(w).cuda())
        x = rng.standard_normal((n, din)).astype(np.float32)
        y = rng.integers(0, classes, n).astype(np.int32)
        ora.step(x, y, 0.5)
        gpu.step(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), 0.5)
        for l in range(2):
            scale = ora.last["max_change_scale"][l]
            assert (scale < 1.0) == (limit < 1.0)
            assert float(gpu.last_max_change_scale(l).item()) == pytest.approx(scale, rel=1.0e-6)
            assert rel(gpu.get_params(l).cpu().numpy(), ora.W[l]) < TOL, l


def test_maximum_change_of_rows_beyond_fp32_squares(ngsgd):
    """Rows whose squares sum to infinity in fp32: the change stays limited, here to nothing.  The large input has no weight, so the
    layer's outputs and derivatives are ordinary."""
    import torch
    n, dims = 70, [8, 40, 9]
    rng = np.random.default_rng(9700)
    weights = random_weights(rng, dims)
    weights[0][:, 2] = 0.0
    x = rng.standard_normal((n, dims[0])).astype(np.float32)
    x[:, 2] = 1.0e20
    y = rng.integers(0, dims[2], n).astype(np.int32)
    for limit in (0.0, 0.1):   # without and with
        gpu = ngsgd.Network(dims, [workloads.TANH], n, rank_in=0, rank_out=0, max_change_per_sample=limit)
        for l, w in enumerate(weights):
            gpu.set_params(l, torch.from_numpy(w).cuda())
        gpu.step(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), 0.5)
        got = gpu.get_params(0).cpu().numpy()
        if limit == 0.0:
            assert np.abs(got[:, 2]).max() > 1.0e18
        else:
            assert float(gpu.last_max_change_scale(0).item()) == 0.0
            assert np.array_equal(got, weights[0])
            assert 0.0 < float(gpu.last_max_change_scale(1).item()) <= 1.0


# two rows to a workgroup; rows longer than it keeps in registers (5120), a last piece of one to three columns, a single row
@pytest.mark.parametrize("N,D,R", [(1, 5, 1), (2, 1025, 3), (3, 5119, 2), (65, 5121, 20), (66, 6002, 33), (129, 10243, 20)])
def test_scaled_rows(ngsgd, N, D, R):
    import torch
    rng = np.random.default_rng(9900 + N + D)
    kw = dict(num_samples_history=600.0, update_period=2, always_update_first=1)
    rows = max(N, R + 2)   # (the first minibatch has more rows than the rank)
    ora = OnlineNaturalGradient(D, R, **kw)
    pre = ngsgd.Preconditioner(D, R, max_batch=rows, **kw)
    for step in range(4):   # with and without an update
        M = data(rng, rows if step == 0 else N, D)
        want, g_o, rn_o = ora.precondition(M)
        got, g_g, rn_g = gpu_call(torch, pre, M, ld=D + (-D) % 4)
        assert rel(got, want) < 1.0e-4, step
        assert g_g == pytest.approx(g_o, rel=1.0e-4)
        assert rel(rn_g, rn_o) < 2.0e-4
