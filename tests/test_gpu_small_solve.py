"""Small least-squares problems, solved by one wavefront each (smallls_kernels.hpp): sizes on both sides of the line to
the panels, many problems, zero pivots, values that are not finite, Newton steps and batches, the workspace."""
import numpy as np
import pytest

import gpu_util as U
import test_gpu_blockls as T
from paper_1402_2626_amd import synth

pytestmark = pytest.mark.gpu

# the largest N * n of the one-wavefront solve, by (level, real)
LINE = {(1, False): 400, (2, False): 150, (4, False): 36, (1, True): 600, (2, True): 400, (4, True): 100}


@pytest.fixture(scope="module")
def pe():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_1402_2626_amd import polyeval
    return polyeval


@pytest.mark.parametrize("L,real", list(LINE))
def test_sizes(pe, L, real):
    """One unknown; square and tall problems at the line; the first beyond it; more rows than lanes."""
    top = LINE[L, real]
    side = int(top ** 0.5)
    for N, n in ((1, 1), (2, 1), (top, 1), (top + 1, 1), (side, side), (side + 1, side), (top // 3, 3), (top // 2, 2)):
        rng = synth.rng_for((501, L, N, n))
        Ab = T._limbs((502, L, N, n), rng.standard_normal((3, 1 if real else 2, N, n + 1)), L)
        x, resid, R, Q = T._solve(pe, Ab)
        for p in (0, 2):
            T._check(Ab[p], x[p], R[p], Q[p], L, rng, count=6)
            lead = Ab[p, :, 0, :, n]
            assert abs(resid[p, 0] - np.sqrt((lead ** 2).sum())) <= 1e-12 * resid[p, 0]
            assert resid[p, 1] == np.abs(x[p, :, 0]).max()


@pytest.mark.parametrize("L,real", list(LINE))
def test_zero_pivots_and_nonfinite(pe, L, real):
    """Among good problems: a column twice, a zero column, a NaN, an infinite right-hand side."""
    import torch
    N, n = 6, 4
    rng = synth.rng_for((511, L))
    Ab = T._limbs((512, L), rng.standard_normal((5, 1 if real else 2, N, n + 1)), L)
    good = T._solve(pe, Ab[:1])
    Ab[1, ..., 2] = Ab[1, ..., 0]
    Ab[2, ..., 1] = 0.0
    Ab[3, 0, 0, 2, 1] = np.nan
    Ab[4, 0, 0, 2, n] = np.inf
    x, resid, R, Q = T._solve(pe, Ab)
    assert np.array_equal(x[0], good[0][0]) and np.array_equal(R[0], good[2][0]) and np.array_equal(Q[0], good[3][0])
    for p, done in ((1, 2), (2, 1), (3, 1)):
        assert resid[p, 1] == -1.0 and not x[p].any()
        assert not R[p][:, :, done:].any() and not Q[p][..., done:].any()
    assert not np.isfinite(x[4]).all() and np.isinf(resid[4, 0])
    # the input is the caller's
    d = U.to_device(Ab)
    before = d.clone()
    pe.lstsq(d)
    torch.cuda.synchronize()
    assert torch.equal(torch.nan_to_num(d), torch.nan_to_num(before))


@pytest.mark.parametrize("L", [1, 2, 4])
def test_newton_batch_and_workspace(pe, L):
    """Newton steps of small systems, alone, at many points and in a batch, against the residual's decrease; no more
    workspace than [J | -F], R and y."""
    import torch
    sizes, P = [(3, 3), (6, 5), (2, 1)], 40
    S, xs = [], []
    for N, n in sizes:
        s = synth.random_system((521, L, N), L, n_vars=n, n_polys=N, m=6, k=min(3, n))
        S.append(pe.System.from_sparse(s))
        xs.append(U.to_device(synth.unit_circle_points(synth.rng_for((522, n)), P, n, L)))
        assert S[-1].newton_workspace_bytes(P) <= P * (16 * L * (N * (n + 1) + n * (n + 2)) + 1024) + 1024
    for t in S[1:]:
        if t.info()["segment"] != S[0].info()["segment"]:
            t.set_shape(0, segment=S[0].info()["segment"])
    B = pe.Batch(S)
    xb, rb = B.newton_step(torch.cat([x.reshape(-1) for x in xs]), P)
    at = 0
    for i, (t, x) in enumerate(zip(S, xs)):
        F, J = t.eval(x)
        y, r = t.newton_step(x.clone())
        z, _ = t.newton_step(x[7:8].clone())
        torch.cuda.synchronize()
        assert torch.equal(y[7:8], z)
        assert torch.equal(xb[at:at + x.numel()], y.reshape(-1)) and torch.equal(rb[i], r)
        at += x.numel()
        lead = lambda a: (a[:, 0].sum(1) + 1j * a[:, 1].sum(1)).cpu().numpy()  # noqa: E731
        A, f, dx = lead(J), lead(F), lead(y) - lead(x)
        for p in range(P):
            want = np.linalg.lstsq(A[p], -f[p], rcond=None)[0]
            assert np.abs(dx[p] - want).max() <= 1e-9 * max(1.0, np.abs(want).max()) * np.linalg.cond(A[p])
    for h in [B] + S:
        h.close()
