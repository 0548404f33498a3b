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
# then shapes whose tile counts select the other tiles (test_kernel_sources.py looks after that)
SHAPES = [(1, 4, 3, 2), (2, 8, 33, 5), (31, 36, 33, 17), (32, 64, 32, 64), (33, 60, 65, 31), (63, 64, 95, 97), (65, 68, 127, 129),
          (96, 128, 191, 193), (129, 256, 257, 63), (200, 300, 1000, 259), (512, 360, 3001, 1009), (515, 1024, 2051, 333),
          (1027, 700, 2050, 301), (300, 2048, 2040, 300), (257, 100, 70, 4957), (291, 112, 61, 4974), (129, 100, 2545, 392), (92, 584, 133, 4882)]


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


def plain_pair(ngsgd, dims, weights, n):
    import torch
    nonlin = [workloads.TANH] * (len(dims) - 2)
    ora = NGSGDNetwork(dims, nonlin, weights, rank_in=0, rank_out=0)
    gpu = ngsgd.Network(dims, nonlin, n, rank_in=0, rank_out=0)
    for l, w in enumerate(weights):
        gpu.set_params(l, torch.from_numpy(w).cuda())
    return ora, gpu


def gradients(ora, gpu, x, y):
    """(oracle, GPU) mean log-probability and gradients of one step."""
    import torch
    with np.errstate(over="ignore", under="ignore"):
        obj = ora.step(x, y, 0.01)
    out = gpu.step(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda(), 0.01)
    grads = [gpu.last_gradient(l).cpu().numpy() for l in range(len(ora.W))]
    return (obj, ora.last["delta"]), (float(out.item()), grads)


@pytest.mark.parametrize("where", ["features", "hidden weights", "output weights"])
def test_operands_near_the_smallest_normal_number(ngsgd, where):
    """Features and weights of about 2^-118: their products keep the precision of any other.  The last layer's gradient
    holds the features (hidden activations) themselves, the first layer's the derivatives behind the output weights."""
    rng = np.random.default_rng(5)
    tiny = np.float32(2.0 ** -118)
    dims = [36, 50] if where == "features" else [36, 40, 50]
    n = 70
    weights = [rng.standard_normal((dims[l + 1], dims[l] + 1)).astype(np.float32) / np.float32(np.sqrt(dims[l] + 1)) for l in range(len(dims) - 1)]
    x = rng.standard_normal((n, 36)).astype(np.float32)
    y = rng.integers(0, 50, n).astype(np.int32)
    if where == "features":
        x *= tiny
    else:
        weights[0 if where == "hidden weights" else 1] *= tiny
    ora, gpu = plain_pair(ngsgd, dims, weights, n)
    (_, want), (_, got) = gradients(ora, gpu, x, y)
    at = 0 if where == "output weights" else len(dims) - 2
    cols = slice(None) if where == "output weights" else slice(0, -1)      # (the bias input is one)
    assert 0.0 < np.linalg.norm(want[at][:, cols]) < 1e-30
    assert rel(got[at][:, cols], want[at][:, cols]) < TOL


def test_largest_finite_feature(ngsgd):
    """A feature within 0.4 % of the largest fp32 number and a weight of zero: only the gradient sees it."""
    rng = np.random.default_rng(6)
    n, din, classes = 90, 36, 40
    x = rng.standard_normal((n, din)).astype(np.float32)
    x[17, 5] = 3.4e38
    y = rng.integers(0, classes, n).astype(np.int32)
    ora, gpu = plain_pair(ngsgd, [din, classes], [np.zeros((classes, din + 1), np.float32)], n)
    (_, want), (_, got) = gradients(ora, gpu, x, y)
    others = [c for c in range(din + 1) if c != 5]
    assert rel(got[0][:, 5], want[0][:, 5]) < TOL
    assert rel(got[0][:, others], want[0][:, others]) < TOL


@pytest.mark.parametrize("where", ["features", "weights"])
@pytest.mark.parametrize("n,din,hidden,classes", SHAPES[2:])
def test_operands_beyond_the_range_of_the_split(ngsgd, n, din, hidden, classes, where):
    """Features (softmax weights) of about 2^106, beyond what the bf16 terms hold, with hidden (softmax) inputs so small that
    the logits are ordinary: every tile of the forward products and of the first layer's gradient (and of the backward
    product) is formed on the fp32 matrix unit, in chains of 128 products: the same error as the split's."""
    rng = np.random.default_rng(n + classes)
    weights = [rng.standard_normal((o, i + 1)).astype(np.float32) / np.float32(np.sqrt(i + 1)) for i, o in ((din, hidden), (hidden, classes))]
    x = rng.standard_normal((n, din)).astype(np.float32)
    if where == "features":
        x *= np.float32(2.0 ** 106)
        weights[0] *= np.float32(2.0 ** -108)
    else:
        weights[0] *= np.float32(2.0 ** -106)
        weights[1][:, :-1] *= np.float32(2.0 ** 106)
    y = rng.integers(0, classes, n).astype(np.int32)
    ora, gpu = plain_pair(ngsgd, [din, hidden, classes], weights, n)
    (obj_o, want), (obj_g, got) = gradients(ora, gpu, x, y)
    assert abs(obj_g - obj_o) < 2e-6 * abs(obj_o) + 1e-6
    for l in range(2):
        assert rel(got[l], want[l]) < TOL, l


@pytest.mark.parametrize("din,hidden,classes", [(36, 40, 50), (128, 300, 259)])
def test_class_with_an_infinite_bias(ngsgd, din, hidden, classes):
    """A class switched off by a bias of minus infinity: it has probability zero, the others share the rest, and it gives
    no derivative."""
    rng = np.random.default_rng(7)
    n, off = 130, 33
    weights = [rng.standard_normal((o, i + 1)).astype(np.float32) / np.float32(np.sqrt(i + 1)) for i, o in ((din, hidden), (hidden, classes))]
    weights[1][off, -1] = -np.inf
    x = rng.standard_normal((n, din)).astype(np.float32)
    y = rng.integers(0, 30, n).astype(np.int32)
    ora, gpu = plain_pair(ngsgd, [din, hidden, classes], weights, n)
    (obj_o, want), (obj_g, got) = gradients(ora, gpu, x, y)
    assert abs(obj_g - obj_o) < 2e-6 * abs(obj_o)
    for l in range(2):
        assert rel(got[l], want[l]) < TOL, l
    assert not got[1][off].any()


@pytest.mark.parametrize("din,classes", [(36, 50), (360, 259)])
def test_product_beyond_the_largest_number(ngsgd, din, classes):
    """A class whose logit is a finite number times a finite number of the other sign, -1.4e50: minus infinity."""
    rng = np.random.default_rng(8)
    n, off = 130, 33
    weights = [rng.standard_normal((classes, din + 1)).astype(np.float32) / np.float32(np.sqrt(din + 1))]
    weights[0][:, 3] = 0.0
    weights[0][off, 3] = -1.3e25
    x = rng.standard_normal((n, din)).astype(np.float32)
    x[:, 3] = rng.uniform(1.0e25, 1.2e25, n).astype(np.float32)
    y = rng.integers(0, 30, n).astype(np.int32)
    ora, gpu = plain_pair(ngsgd, [din, classes], weights, n)
    (obj_o, want), (obj_g, got) = gradients(ora, gpu, x, y)
    assert abs(obj_g - obj_o) < 2e-6 * abs(obj_o)
    others = [c for c in range(din + 1) if c != 3]
    assert rel(got[0][:, 3], want[0][:, 3]) < TOL
    assert rel(got[0][:, others], want[0][:, others]) < TOL
    assert not got[0][off].any()


# One product forms its sums with a relative error (2-norm) of at most 2.5e-7: 1.1e-7 to 1.6e-7 measured for the update, the
# only product of its gradient.  The others' gradients have a short second product and element-wise parts on top, together
# less than another 2.5e-7: 1.7e-7 to 2.5e-7 measured.  (Chains of fp32 matrix instructions: up to 1.7e-6.)
@pytest.mark.parametrize("k", [301, 2049, 8000])
@pytest.mark.parametrize("which", ["forward", "backward", "update"])
def test_precision_of_one_product(ngsgd, which, k):
    """The length of the sum of one product grows, the other products of the gradient are short or exact."""
    rng = np.random.default_rng(k)
    n, din, hidden, classes = 64, 64, 96, 64
    if which == "update":                       # O^T X over k rows; O is one-hot minus 1/64, exact
        n, dims = k, [din, classes]
        weights = [np.zeros((classes, din + 1), np.float32)]
    elif which == "forward":                    # tanh(a) = a for |a| of 2^-14; the softmax layer is zero: O as above
        dims = [(k + 2) // 4 * 4, hidden, classes]
        weights = [(rng.standard_normal((hidden, dims[0] + 1)) * 2.0 ** -20).astype(np.float32), np.zeros((classes, hidden + 1), np.float32)]
    else:                                       # O W over k classes, the hidden layer is zero: derivatives pass unchanged
        dims = [din, hidden, k]
        weights = [np.zeros((hidden, din + 1), np.float32), (rng.standard_normal((k, hidden + 1))).astype(np.float32)]
        weights[1][:, -1] = 0.0
    x = rng.standard_normal((n, dims[0])).astype(np.float32)
    y = rng.integers(0, dims[-1], n).astype(np.int32)
    ora, gpu = plain_pair(ngsgd, dims, weights, n)
    (_, want), (_, got) = gradients(ora, gpu, x, y)
    at = 1 if which == "forward" else 0
    cols = slice(0, -1) if which == "forward" else slice(None)
    err = rel(got[at][:, cols], want[at][:, cols])
    print(which, k, err)
    assert err < (2.5e-7 if which == "update" else 5e-7)
