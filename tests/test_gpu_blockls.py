"""The least-squares solve in panels (blockls_kernels.hpp) at the sizes where
its tiles end: panels of 32 complex or 64 real columns, chunks of 64 rows,
sub-blocks of the back substitution, groups of problems; and the matrices its
panels treat specially (columns and rows of very different size, panels too
ill-conditioned for their Gram matrix, zero pivots, values that are not
finite)."""
import numpy as np
import pytest

import gpu_util as U
import oracle as O
from paper_1402_2626_amd import synth

pytestmark = pytest.mark.gpu

UNIT = {1: 2.0 ** -53, 2: 2.0 ** -104, 4: 2.0 ** -206}


@pytest.fixture(scope="module")
def pe():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_1402_2626_amd import polyeval
    return polyeval


def _limbs(seed, lead, L):
    """[P, C, N, n + 1] leading limbs with random limbs below: [P, C, L, N, n + 1]."""
    return np.ascontiguousarray(np.moveaxis(synth.lower_limbs(synth.rng_for(seed), lead, L), 0, 2))


def _num(a, *idx):
    im = a[(1, slice(None)) + idx] if a.shape[0] == 2 else np.zeros(a.shape[1])
    return O.cdy_from_limbs(a[(0, slice(None)) + idx], im)


def _solve(pe, Ab):
    import torch
    x, resid, R, Q = pe.lstsq(U.to_device(Ab), want_R=True, want_Q=True)
    torch.cuda.synchronize()
    return [t.cpu().numpy() for t in (x, resid, R, Q)]


def _check(Ab, x, R, Q, L, rng, count=10):
    """Exactly from the limbs, on sampled entries: A = QR (within 64 N u of the
    sum of the absolute products), Q^H Q = I (Gram-Schmidt keeps it to u times
    the condition number at worst), R x = y (within 64 n u of the absolute
    products), with the bounds of the least-squares tests."""
    N, n = Q.shape[2], Q.shape[3]
    u = UNIT[L]
    lead = Ab[0, 0] + 1j * (Ab[1, 0] if Ab.shape[0] == 2 else 0)
    scale = np.linalg.norm(lead[:, :n], axis=0)
    s = np.linalg.svd(lead[:, :n] / scale, compute_uv=False)
    kappa = s[0] / s[-1]
    if kappa > 1e14:
        kappa = 1e3 / u ** 0.5 if L == 1 else 1e30  # beyond what 64 bits can say
    pick = lambda k: sorted({0, k - 1, *(int(v) for v in rng.integers(k, size=count))})  # noqa: E731
    for i in pick(N)[:4]:
        for j in pick(n)[:5]:
            acc, mag = O.ZERO, 0.0
            for k in range(j + 1):
                q, r = _num(Q, i, k), _num(R, k, j)
                acc = O.cdy_add(acc, O.cdy_mul(q, r))
                mag += O.cdy_abs_float(q) * O.cdy_abs_float(r)
            d = O.cdy_abs_float(O.cdy_add(_num(Ab, i, j), O.cdy_neg(acc)))
            assert d <= 64 * N * u * mag, ("A - QR", i, j, d / (mag * u))
    for k in pick(n)[:4]:
        for m in pick(n)[-4:]:
            acc = O.ZERO
            for i in range(N):
                acc = O.cdy_add(acc, O.cdy_mul(O.cdy_conj(_num(Q, i, k)), _num(Q, i, m)))
            if k == m:
                acc = O.cdy_add(acc, (-1, 0, 0))
            assert O.cdy_abs_float(acc) <= 64 * N * u * kappa, ("Q^H Q - I", k, m, O.cdy_abs_float(acc) / u, kappa)
    for k in pick(n)[:6]:
        acc, mag = O.cdy_neg(_num(R, k, n)), O.cdy_abs_float(_num(R, k, n))
        for j in range(k, n):
            r, v = _num(R, k, j), _num(x, j)
            acc = O.cdy_add(acc, O.cdy_mul(r, v))
            mag += O.cdy_abs_float(r) * O.cdy_abs_float(v)
        assert O.cdy_abs_float(acc) <= 64 * n * u * mag, ("R x - y", k, O.cdy_abs_float(acc) / (mag * u))
    low = np.tril(np.ones((n, n)), -1) > 0
    assert np.all(R[:, :, :, :n][:, :, low] == 0.0)
    assert np.all(np.diagonal(R[0, 0]) > 0.0)


@pytest.mark.parametrize("L, real, N, n", [
    (2, False, 1, 1), (2, False, 64, 32), (2, False, 65, 33), (2, False, 97, 64), (1, False, 130, 65),
    (4, False, 63, 31), (4, False, 70, 33), (1, True, 66, 65), (2, True, 64, 63), (2, True, 129, 128),
    (4, True, 68, 65), (2, False, 290, 257)])
def test_edges_of_panels(pe, L, real, N, n):
    """Sizes one below, at and one above a panel, a chunk and a block."""
    rng = synth.rng_for((911, L, N, n))
    Ab = _limbs((912, L, N, n), rng.standard_normal((2, 1 if real else 2, N, n + 1)), L)
    x, resid, R, Q = _solve(pe, Ab)
    for p in range(2):
        _check(Ab[p], x[p], R[p], Q[p], L, rng)
        lead = Ab[p, :, 0, :, n]
        assert abs(resid[p, 0] - np.sqrt((lead ** 2).sum())) <= 1e-12 * resid[p, 0]
        assert resid[p, 1] == np.abs(x[p, :, 0]).max()


@pytest.mark.parametrize("L", [1, 2, 4])
@pytest.mark.parametrize("what", ["columns", "rows", "near", "hilbert", "triangular"])
def test_uneven_and_ill_conditioned(pe, L, what):
    """Columns over 30 (rows over 3) orders of magnitude; columns that agree
    to 1e-6 and 1e-11 with others of their panel (too close for the Gram
    matrix, so that the panel is orthogonalised column by column), a Hilbert
    matrix of condition 1e16 (orthogonalised twice); a triangular matrix with
    a strong diagonal."""
    rng = synth.rng_for((921, L))
    N, n, C = 80, 50, 2
    a = rng.standard_normal((1, C, N, n + 1))
    if what == "columns":
        a *= 10.0 ** (-(10 if L == 1 else 30) * rng.random((1, 1, 1, n + 1)))
    elif what == "rows":
        a *= 10.0 ** (-3 * rng.random((1, 1, N, 1)))
    elif what == "near":
        a[:, :, :, 17] = a[:, :, :, 5] + 1e-6 * a[:, :, :, 17]
        if L > 1:
            a[:, :, :, 45] = a[:, :, :, 33] + 1e-11 * a[:, :, :, 45]
    elif what == "hilbert":
        m = 6 if L == 1 else 12
        i = np.arange(N)
        a = np.concatenate([1.0 / (i[:, None] + i[None, :m] + 1.0), np.ones((N, 1))], 1)[None, None]
    else:
        a = np.triu(a)
        a[0, 0, np.arange(n), np.arange(n)] = 20.0
    Ab = _limbs((922, L), a, L)
    x, resid, R, Q = _solve(pe, Ab)
    assert resid[0, 1] > 0.0
    _check(Ab[0], x[0], R[0], Q[0], L, rng)


@pytest.mark.parametrize("L, real", [(1, False), (2, False), (4, True)])
def test_zero_pivots_and_values_not_finite(pe, L, real):
    """Repeated and zero columns (in the first and in a later panel) and
    columns that are not finite flag their problem alone; a right-hand side
    that is not finite gives a solution that is not."""
    C = 1 if real else 2
    N, n, P = 90, 80, 7
    rng = synth.rng_for((931, L))
    Ab = _limbs((932, L), rng.standard_normal((P, C, N, n + 1)), L)
    Ab[1, ..., 9] = Ab[1, ..., 4]
    Ab[2, ..., 75] = Ab[2, ..., 3]
    Ab[3, ..., 70] = 0.0
    Ab[4, 0, 0, 5, 66] = np.nan
    Ab[5, 0, 0, 7, 2] = np.inf
    Ab[6, 0, 0, 11, n] = np.nan
    x, resid, R, Q = _solve(pe, Ab)
    assert np.isfinite(x[0]).all() and resid[0, 1] > 0.0
    for p in range(1, 6):
        assert resid[p, 1] == -1.0 and np.all(x[p] == 0.0), p
    assert not np.isfinite(x[6][0, 0]).any() and resid[6, 1] >= 0.0
    _check(Ab[0], x[0], R[0], Q[0], L, rng, 4)


def test_more_problems_than_slots(pe):
    """12000 problems of 5 x 3 in double: more than go through at once."""
    import torch
    P, N, n = 12000, 5, 3
    rng = synth.rng_for(941)
    a = rng.standard_normal((P, 2, N, n + 1))
    x, resid, _, _ = pe.lstsq(U.to_device(np.ascontiguousarray(a[:, :, None])))
    torch.cuda.synchronize()
    z = a[:, 0] + 1j * a[:, 1]
    A, b = z[:, :, :n], z[:, :, n]
    q, r = np.linalg.qr(A)
    want = np.linalg.solve(r, np.einsum("pij,pi->pj", q.conj(), b)[..., None])[..., 0]
    got = x.cpu().numpy()
    got = got[:, 0, 0] + 1j * got[:, 1, 0]
    kappa = np.linalg.cond(A)
    err = np.abs(got - want).max(1) / np.abs(want).max(1)
    assert np.all(err <= 10 * N * kappa ** 2 * 2.0 ** -53), np.max(err / kappa ** 2)


def test_solve_graph_replay(pe):
    """A captured solve of several panels and of a panel orthogonalised column
    by column, replayed with eager work between the replays."""
    import torch
    rng = synth.rng_for(951)
    a = rng.standard_normal((2, 2, 150, 101))
    a[1, :, :, 40] = a[1, :, :, 34] + 1e-11 * a[1, :, :, 40]
    Ab = U.to_device(_limbs(952, a, 2))
    nbytes = pe._lib.pe_lstsq_workspace_bytes(2, 2, 150, 100)
    ws = torch.empty((nbytes + 7) // 8, dtype=torch.float64, device="cuda")
    want = [t.clone() for t in pe.lstsq(Ab, workspace=ws)[:2]]
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    pe.lstsq(Ab, workspace=ws, stream=s)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        x, resid, _, _ = pe.lstsq(Ab, workspace=ws, stream=s)
    for _ in range(3):
        x.zero_()
        ws.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(x, want[0]) and torch.equal(resid, want[1])
