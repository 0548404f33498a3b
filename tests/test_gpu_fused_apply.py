"""GPU parity of the fused apply path (calls that do not update their factor, App. B.5 "without updating"):
ngsgd_precondition through the C ABI against the float64 oracle on the same seeded inputs.

The fused kernel lets the workgroups of a block of 64 rows wait for each other's share of H = X W^T; the wait is
bounded and a workgroup that gives up forms its H rows itself.  Both routes are held to the same bar (1e-4 relative
Frobenius): the ordinary one, and the slow one forced from the host with a wait limit of zero.
"""
import numpy as np
import pytest

import workloads
from oracle.online_ng import OnlineNaturalGradient

pytestmark = pytest.mark.gpu

TOL = 1.0e-4


def rel(a, b):
    return float(np.linalg.norm(np.asarray(a, np.float64) - np.asarray(b, np.float64)) /
                 max(np.linalg.norm(np.asarray(b, np.float64)), 1e-300))


def data(rng, N, D, decay=0.97, mean=0.3):
    scales = decay ** np.arange(D) + 0.02
    x = rng.standard_normal((N, D)) * scales[None, :] + mean * np.sin(np.arange(D))[None, :]
    return x[:, rng.permutation(D)].astype(np.float32)


def gpu_call(torch, pre, M, ld):
    N, D = M.shape
    buf = torch.full((N, ld), 777.0, dtype=torch.float32, device="cuda")   # padding holds garbage on purpose
    buf[:, :D] = torch.from_numpy(M).cuda()
    gamma = torch.zeros(1, dtype=torch.float32, device="cuda")
    rn2 = torch.zeros(N, dtype=torch.float32, device="cuda")
    pre.precondition(buf, gamma, rn2)
    torch.cuda.synchronize()
    out = buf.cpu().numpy()
    if ld > D:
        assert np.all(out[:, D:] == 777.0), "columns beyond dim must not be touched"
    return out[:, :D], float(gamma.item()), rn2.cpu().numpy()


SHAPES = [(100, 333, 7), (64, 160, 1), (65, 161, 33), (129, 40, 4), (300, 1000, 96), (37, 50, 20), (200, 3001, 20),
          (256, 640, 80), (90, 2000, 81)]


@pytest.mark.parametrize("wait_us", [2000, 0])
@pytest.mark.parametrize("N,D,R", SHAPES)
def test_calls_without_update_match_oracle(ngsgd, N, D, R, wait_us):
    """Schedule: calls 0, 1 update (always_update_first = 2), 2 and 3 apply only, 4 updates, 5..7 apply only; the
    apply-only calls take the fused kernel.  Rows vary (fewer rows than the first call, a single row)."""
    import torch
    rng = np.random.default_rng(7000 + 13 * N + D + R)
    kw = dict(num_samples_history=600.0, update_period=4, always_update_first=2)
    ora = OnlineNaturalGradient(D, R, **kw)
    pre = ngsgd.Preconditioner(D, R, max_batch=N, **kw)
    ngsgd.set_wait_limit_us(wait_us)
    try:
        for step in range(8):
            n = {3: max(1, N - 9), 6: 1}.get(step, N)
            M = data(rng, n, D)
            print(f"fused apply case N={n} D={D} R={R} step={step} wait_us={wait_us}", flush=True)
            expect, g_o, rn_o = ora.precondition(M)
            got, g_g, rn_g = gpu_call(torch, pre, M, ld=D + (-D) % 4 + (8 if step % 2 else 0))
            assert rel(got, expect) < TOL, f"step {step}"
            assert g_g == pytest.approx(g_o, rel=1e-4)
            assert rel(rn_g, rn_o) < 2e-4
            assert abs(np.linalg.norm(got.astype(np.float64)) / np.linalg.norm(M.astype(np.float64)) - 1.0) < 1e-5
    finally:
        ngsgd.set_wait_limit_us(2000)


@pytest.mark.parametrize("which", ["input", "output"])
def test_c2_full_size_without_update(ngsgd, which):
    """BASELINE configs[2] shapes at full size, apply-only calls between periodic updates."""
    import torch
    spec = workloads.c2_input_side() if which == "input" else workloads.c2_output_side()
    kw = dict(num_samples_history=spec.num_samples_history, update_period=4, always_update_first=3)
    ora = OnlineNaturalGradient(spec.dim, spec.rank, **kw)
    pre = ngsgd.Preconditioner(spec.dim, spec.rank, max_batch=spec.rows, **kw)
    ld = (spec.dim + 3) // 4 * 4
    for step in range(8):
        print(f"fused apply full size {spec.name} step={step}", flush=True)
        M = workloads.spectrum_matrix(spec, step)
        expect, g_o, rn_o = ora.precondition(M)
        got, g_g, rn_g = gpu_call(torch, pre, M, ld)
        assert rel(got, expect) < TOL, f"step {step}"
        assert g_g == pytest.approx(g_o, rel=1e-4)
        assert rel(rn_g, rn_o) < 2e-4


# 1024 patches of 64 x 160 (ceil(N / 64) * ceil(D / 160)), the fewest for wide ones and the most of one matrix.  Four of these go
# wide: the last patch of 320 columns has four pieces of 64 and one column, 201 columns, 161 (two pieces and 33), all; the last row
# block one row, a few, all.  The others would leave dies idle and stay narrow.
WIDE = [(8129, 1121, 80), (8192, 1280, 33), (4033, 2497, 41), (1990, 5001, 96), (65473, 129, 81), (4096, 2401, 80), (4090, 2560, 33)]


@pytest.mark.parametrize("N,D,R", WIDE)
def test_wide_patches_match_oracle(ngsgd, N, D, R):
    import torch
    rng = np.random.default_rng(8000 + N + D + R)
    kw = dict(num_samples_history=4000.0, update_period=4, always_update_first=1)
    ora = OnlineNaturalGradient(D, R, **kw)
    pre = ngsgd.Preconditioner(D, R, max_batch=N, **kw)
    try:
        for step, wait_us in enumerate([2000, 2000, 0]):   # one update, one call as it should go, one that leaves patches over
            ngsgd.set_wait_limit_us(wait_us)
            M = data(rng, N, D)
            print(f"wide patches N={N} D={D} R={R} step={step} wait_us={wait_us}", flush=True)
            expect, g_o, rn_o = ora.precondition(M)
            got, g_g, rn_g = gpu_call(torch, pre, M, ld=D + (-D) % 4)
            assert rel(got, expect) < TOL, f"step {step}"
            assert g_g == pytest.approx(g_o, rel=1e-4)
            assert rel(rn_g, rn_o) < 2e-4
    finally:
        ngsgd.set_wait_limit_us(2000)


def test_deferred_patches_are_shared_by_the_workgroups(ngsgd):
    """A call that leaves all of its patches to the finishing kernel: 0.4 ms for 512 x 5000 with all of the chip, 84 when one
    workgroup is left to do it."""
    import torch
    N, D, R = 512, 5000, 80
    rng = np.random.default_rng(7700)
    pre = ngsgd.Preconditioner(D, R, max_batch=N, update_period=1000, always_update_first=1)
    M = data(rng, N, D)
    gpu_call(torch, pre, M, ld=D)
    buf, gamma, rn2 = torch.from_numpy(M).cuda().contiguous(), torch.zeros(1, device="cuda"), torch.zeros(N, device="cuda")
    start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    ngsgd.set_wait_limit_us(0)
    try:
        times = []
        for _ in range(5):
            start.record()
            pre.precondition(buf, gamma, rn2)
            end.record()
            torch.cuda.synchronize()
            times.append(start.elapsed_time(end))
    finally:
        ngsgd.set_wait_limit_us(2000)
    assert min(times) < 5.0, times


@pytest.mark.parametrize("N,D,R", [(300, 1000, 33), (65, 161, 5)])
def test_captured_call_that_leaves_patches_over(ngsgd, N, D, R):
    """A captured call whose patches are all deferred, replayed between eager calls that defer none and some that do."""
    import torch
    rng = np.random.default_rng(7800 + N)
    kw = dict(max_batch=N, num_samples_history=600.0, update_period=1 << 30, always_update_first=1)
    plain, captured = ngsgd.Preconditioner(D, R, **kw), ngsgd.Preconditioner(D, R, **kw)
    ld = D + (-D) % 4
    static, gamma, rn2 = torch.zeros(N, ld, device="cuda"), torch.zeros(1, device="cuda"), torch.zeros(N, device="cuda")
    graph = torch.cuda.CUDAGraph()

    def matrix():
        return torch.nn.functional.pad(torch.from_numpy(np.ascontiguousarray(data(rng, N, D))), (0, ld - D)).cuda()

    def both(replay, wait_us=2000):
        m = matrix()
        static.copy_(m)
        plain.precondition(m[:, :D])
        if replay:
            graph.replay()
        else:
            ngsgd.set_wait_limit_us(wait_us)
            captured.precondition(static[:, :D], gamma, rn2)
            ngsgd.set_wait_limit_us(2000)
        torch.cuda.synchronize()
        want, got = m[:, :D].cpu().numpy(), static[:, :D].cpu().numpy()
        assert rel(got, want) < 1e-5
        # squared row norms of what came out: fp32 sums of squares, 1e-5 covers them
        assert rel(rn2.cpu().numpy(), (got.astype(np.float64) ** 2).sum(1)) < 1e-5

    try:
        m = matrix()                 # the update, the same for both
        static.copy_(m)
        plain.precondition(m[:, :D])
        captured.precondition(static[:, :D], gamma, rn2)
        both(False)
        ngsgd.set_wait_limit_us(0)
        with torch.cuda.graph(graph):
            captured.precondition(static[:, :D], gamma, rn2)
        ngsgd.set_wait_limit_us(2000)
        for replay, wait_us in ((True, 0), (True, 0), (False, 2000), (True, 0), (False, 0), (False, 2000), (True, 0)):
            both(replay, wait_us)
    finally:
        ngsgd.set_wait_limit_us(2000)
