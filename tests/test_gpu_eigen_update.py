"""GPU parity of the R x R update at the edges of its kernels' tiles, and where the direct eigen-solver hands over to Jacobi."""
import math

import numpy as np
import pytest

from oracle.online_ng import OnlineNaturalGradient, smoothing_and_scales
from test_gpu_precondition import TOL, compare_states, data, gpu_call, rel, upload_state

pytestmark = pytest.mark.gpu


def orthogonality(pre, alpha, D):
    """Largest |W W^T - E| over sqrt(E_ii E_jj) (App. B.3.1)."""
    W, d, rho, _ = pre.get_state()
    W, d = W.cpu().numpy().astype(np.float64), d.cpu().numpy()
    _, e = smoothing_and_scales(d, rho, alpha, D)
    return float(np.abs(W @ W.T / np.sqrt(np.outer(e, e)) - np.eye(len(e))).max())


@pytest.mark.parametrize("R", [1, 2, 3, 4, 15, 16, 17, 18, 19, 31, 32, 33, 34, 35, 47, 48, 49, 63, 64, 65, 79, 80, 81, 95, 96])
def test_update_at_the_edges_of_its_tiles(ngsgd, R):
    """16 columns a stage, one kernel up to rank 32, tiles for ranks up to 48, 80 and 96, four reflections at a time."""
    import torch
    N, D = 140, 260
    rng = np.random.default_rng(9100 + R)
    kw = dict(num_samples_history=500.0, update_period=1)
    ora = OnlineNaturalGradient(D, R, **kw)
    ora.precondition(data(rng, N, D))
    pre = ngsgd.Preconditioner(D, R, max_batch=N, **kw)
    upload_state(torch, pre, ora)
    for _ in range(3):
        M = data(rng, N, D)
        expect, g_o, rn_o = ora.precondition(M)
        got, g_g, rn_g = gpu_call(torch, pre, M)
        assert rel(got, expect) < TOL
        assert rel(rn_g, rn_o) < 2e-4
    compare_states(torch, pre, ora, rng)
    # fp32 rows of J and W: 2^-24 times the square root of the eigenvalues' span, here below 1e4
    assert orthogonality(pre, ora.alpha, D) < 2e-5


@pytest.mark.parametrize("kind", ["equal", "one cluster", "graded", "equal pairs"])
@pytest.mark.parametrize("R", [6, 20, 32, 33, 48, 80, 96])
def test_eigenvalues_that_the_direct_solver_leaves_to_jacobi(ngsgd, R, kind):
    """Rows that do not meet the factor leave Z_t diagonal: with equal eigenvalues (the vectors of a tridiagonal matrix that is
    diagonal are not told apart), or with a span beyond the direct solver's limit.  Jacobi ends after one sweep there, which is
    what the direct solver reports as well; rows that couple the factor's rows by pairs, all alike, leave two eigenvalues, each many
    times, and take rotations."""
    import torch
    N, D = 130, 300
    rng = np.random.default_rng(9200 + R)
    kw = dict(num_samples_history=700.0, update_period=1)
    ora = OnlineNaturalGradient(D, R, **kw)
    ora.precondition(data(rng, N, D))
    ora.R = np.eye(R, D)
    ora.d = {"equal": np.full(R, 0.5), "one cluster": np.where(np.arange(R) < R // 2, 0.5, 0.25 / (1.0 + np.arange(R))),
             "graded": 10.0 ** (-14.0 * np.arange(R) / (R - 1)), "equal pairs": np.full(R, 0.5)}[kind]
    ora.rho = 1e-9
    pre = ngsgd.Preconditioner(D, R, max_batch=N, **kw)
    upload_state(torch, pre, ora)
    M = data(rng, N, D)
    M[:, :R] = 0.0
    if kind == "equal pairs":
        for k in range(R // 2):
            M[k, 2 * k] = M[k, 2 * k + 1] = 12.0
    expect, g_o, _ = ora.precondition(M)
    got, g_g, _ = gpu_call(torch, pre, M)
    assert rel(got, expect) < TOL
    flags, sweeps = pre.diagnostics()
    assert flags & 8 == 0 and (2 if kind == "equal pairs" else 1) <= sweeps <= 20
    compare_states(torch, pre, ora, rng)
    # the rows stay what they were, rounded to fp32; by pairs they mix, as in test_update_at_the_edges_of_its_tiles
    assert orthogonality(pre, ora.alpha, D) < (2e-5 if kind == "equal pairs" else 2e-6)
    M = data(rng, N, D)
    expect, g_o, _ = ora.precondition(M)
    got, g_g, _ = gpu_call(torch, pre, M)
    assert rel(got, expect) < TOL


@pytest.mark.parametrize("R", [5, 20, 32, 33, 48, 80, 96])
def test_graded_factors_in_any_order(ngsgd, R):
    """Eigenvalues over eight decades that do not descend along the rows of the factor, and rows of the minibatch graded alike: the
    update sorts such a matrix, and writes the factor as the order was."""
    import torch
    N, D = 200, 300
    rng = np.random.default_rng(9300 + R)
    kw = dict(num_samples_history=700.0, update_period=1)
    ora = OnlineNaturalGradient(D, R, **kw)
    ora.precondition(data(rng, N, D))
    ora.R = np.eye(R, D)
    ora.d = rng.permutation(10.0 ** (-8.0 * np.arange(R) / (R - 1)))
    ora.rho = 1e-10
    pre = ngsgd.Preconditioner(D, R, max_batch=N, **kw)
    upload_state(torch, pre, ora)
    scale = ora.d.copy()
    for step in range(2):
        M = (rng.standard_normal((N, D)) * 1e-4).astype(np.float32)
        M[:, :R] = (rng.standard_normal((N, R)) * np.sqrt(scale)).astype(np.float32)
        expect, g_o, _ = ora.precondition(M)
        got, g_g, _ = gpu_call(torch, pre, M)
        assert rel(got, expect) < TOL, step
        assert g_g == pytest.approx(g_o, rel=1e-4)
    flags, sweeps = pre.diagnostics()
    # (eigenvalues that meet by chance may still be left to Jacobi: at rank 96 the gaps are a fifth of their size)
    assert flags & 8 == 0 and 1 <= sweeps <= 20


def wells(R, gap, N, D, S):
    """A factor whose D_t falls and rises again the same way, and a minibatch that couples neighbouring rows of it: Z_t has pairs of
    eigenvalues, one vector of each even and one odd, the closer the larger they are.  The coupling is chosen for the closest pair to
    have about the relative distance `gap`."""
    eta = 1.0 - math.exp(-N / S)
    i = np.arange(R)
    d, rho = 0.05 + np.abs(i - 0.5 * (R - 1)) / R, 0.01

    def eigenvalues(coupling):
        M = np.zeros((N, D), np.float32)
        M[i[:-1], i[:-1]] = M[i[:-1], i[1:]] = np.float32(coupling)
        x = M[:, :R].astype(np.float64)
        return M, np.linalg.eigvalsh((1.0 - eta) * np.diag(d + rho) + eta / N * (x.T @ x)) ** 2

    low, high = 0.0, 40.0
    for _ in range(40):
        coupling = 0.5 * (low + high)
        M, c = eigenvalues(coupling)
        low, high = (coupling, high) if (c[-1] - c[-2]) / c[-1] < gap else (low, coupling)
    return M, d, rho


@pytest.mark.parametrize("R", [6, 20, 31, 33, 48, 65, 80, 96])
def test_pairs_of_eigenvalues_around_the_limit_of_the_direct_solver(ngsgd, R):
    """The vectors of a pair get worse as its gap closes: from orthogonal to working precision to not told apart.  The check
    behind the direct solver draws a line in between, and all workgroups of an update have to draw the same.  An ordinary
    update in front of each leaves other rows in the scratch, which a workgroup that dropped out would leave as they are."""
    import torch
    N, D, S = 210, 300, 700.0
    rng = np.random.default_rng(9400 + R)
    kw = dict(num_samples_history=S, update_period=1)
    ora = OnlineNaturalGradient(D, R, **kw)
    ora.precondition(data(rng, N, D))
    pre = ngsgd.Preconditioner(D, R, max_batch=N, **kw)
    served = []
    for k in range(32):
        ora.R, ora.d, ora.rho = np.eye(R, D), np.linspace(1.0, 0.2, R), 0.01
        upload_state(torch, pre, ora)
        M = data(rng, N, D)
        ora.precondition(M)
        gpu_call(torch, pre, M)
        M, ora.d, ora.rho = wells(R, 10.0 ** (-15.0 + 0.25 * k), N, D, S)
        ora.R = np.eye(R, D)
        upload_state(torch, pre, ora)
        expect, g_o, _ = ora.precondition(M)
        got, g_g, _ = gpu_call(torch, pre, M)
        assert rel(got, expect) < TOL, k
        flags, sweeps = pre.diagnostics()
        assert flags & 8 == 0, k
        served.append(sweeps == 1)
        compare_states(torch, pre, ora, rng)
        assert orthogonality(pre, ora.alpha, D) < 2e-5, k   # as in test_update_at_the_edges_of_its_tiles
    print("served by the direct solver, gaps of 1e-15 and up:", "".join("01"[s] for s in served))
    assert served[-1] and not all(served)   # Jacobi rotates such a matrix for several sweeps; the direct solver reports one
