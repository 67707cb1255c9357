"""Evaluation through monomial values (value_kernels.hpp): the structures and points at which it branches,
against the exact oracle and against the reverse sweep.

A system is evaluated through its values only if its occurrences number at least 2 N n; the same monomials
over more variables, the new ones unused, take the reverse sweep, so the two paths can be compared.  The tolerance is
the one of the other evaluation tests."""
import numpy as np
import pytest

import gpu_util as U
from paper_1402_2626_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pe():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_1402_2626_amd import polyeval
    return polyeval


def ragged(seed, level, n, mons, kmax, emax, real):
    """Polynomial p with mons[p] monomials of 0 to kmax variables (most of them kmax)."""
    rng = synth.rng_for(seed)
    k = np.where(rng.random(sum(mons)) < 0.8, kmax, rng.integers(0, kmax + 1, size=sum(mons)))
    var = [np.sort(rng.choice(n, size=int(q), replace=False)) for q in k]
    coef = synth.unit_circle(rng, len(k), level)
    if real:
        coef[1] = 0.0
    return synth.PolySystem(
        level=level, n_vars=n, poly_ptr=np.concatenate([[0], np.cumsum(mons)]).astype(np.int64),
        mon_ptr=np.concatenate([[0], np.cumsum(k)]).astype(np.int64), var_idx=np.concatenate(var).astype(np.int32),
        exps=rng.integers(1, emax + 1, size=int(k.sum())).astype(np.int32), coef=coef)


def widened(s, n):
    return synth.PolySystem(level=s.level, n_vars=n, poly_ptr=s.poly_ptr, mon_ptr=s.mon_ptr, var_idx=s.var_idx,
                            exps=s.exps, coef=s.coef)


def load(pe, s, real):
    if not real:
        return pe.System.from_sparse(s)
    return pe.System(pe.PE_REAL | s.level, s.n_vars, s.poly_ptr, s.mon_ptr, s.var_idx, s.exps,
                     np.ascontiguousarray(s.coef[:1]))


def evaluate(pe, s, x, real, want_J=True):
    """F, J (imaginary parts 0 for real systems) at the points x[P, 2, L, n]."""
    import torch
    S = load(pe, s, real)
    F, J = S.eval(U.to_device(x[:, :1] if real else x), want_J=want_J)
    torch.cuda.synchronize()
    S.close()
    full = lambda t: None if t is None else np.concatenate([t, np.zeros_like(t)], 1) if real else t  # noqa: E731
    return full(F.cpu().numpy()), full(None if J is None else J.cpu().numpy())


def points(seed, P, n, L, real):
    x = synth.unit_circle_points(synth.rng_for(seed), P, n, L)
    if real:  # no small values
        x[:, 1] = 0.0
        x[:, 0] = np.where(np.abs(x[:, 0, :1]) < 0.3, 0.0, x[:, 0])
        x[:, 0, 0] = np.where(x[:, 0, 0] == 0.0, 0.75, x[:, 0, 0])
    return x


def check(s, x, F, J, rows):
    tol = U.tolerance(s)
    eF, eJ = U.max_errors_rows(s, x, F, J, rows, parallel=False)
    U.flush(f"L={s.level} n={s.n_vars}: F {eF:.2e}, J {eJ:.2e} (tolerance {tol:.1e})")
    assert eF <= tol and eJ <= tol, (eF, eJ, tol)


# mons: monomials of each polynomial.  32 KB of values are one block: 2048 complex doubles, 1024 complex double
# doubles, 512 complex quad doubles, twice as many real ones
SHAPES = [
    (1, False, 40, [2047, 0, 1, 2048, 2049, 4100], 6, 2),
    (1, True, 33, [4096, 4097, 300, 1], 5, 3),
    (2, False, 64, [1023, 1024, 1025, 0, 65, 64, 63, 1], 6, 4),
    (2, False, 300, [300] * 5, 13, 1),       # two lanes per monomial
    (2, False, 9, [40] * 7, 7, 2),            # one partly filled slice
    (2, True, 65, [2048, 2049, 1, 128], 5, 3),
    (4, False, 65, [511, 512, 513, 1, 0], 5, 2),
    (4, False, 16, [17] * 4, 6, 3),
    (4, True, 128, [1024, 1030, 3], 8, 2),
    (4, False, 200, [65] * 3, 150, 1),        # sixteen lanes per monomial
    # the table holds x alone: one block, several, a whole row of more values than a block has
    (2, False, 900, [300, 250], 10, 4),
    (4, False, 600, [700, 1, 400], 12, 3),
    (4, False, 1000, [900, 700], 8, 2),
    (4, True, 1900, [1500, 1400], 8, 3),
]


@pytest.mark.parametrize("L,real,n,mons,kmax,emax", SHAPES)
def test_blocks_units_slices(pe, L, real, n, mons, kmax, emax):
    """Edges of blocks, units and slices; F and J of every row, at two points, F alone with the same bits."""
    s = ragged((31, n, L), L, n, mons, kmax, emax, real)
    x = points((32, n), 2, n, L, real)
    F, J = evaluate(pe, s, x, real)
    F1, _ = evaluate(pe, s, x, real, want_J=False)
    assert np.array_equal(F, F1)
    rows = [p for p, m in enumerate(mons) if m <= 300] + [int(np.argmax(mons))]
    check(s, x[1], F[1], J[1], rows)
    # every entry of the first point against the reverse sweep
    wide = 4 * n + s.nnz // max(1, len(mons))
    xw = np.concatenate([x[:1], np.zeros((1, 2, L, wide - n))], 3)
    Fw, Jw = evaluate(pe, widened(s, wide), xw, real)
    assert not Jw[..., n:].any()
    size = np.diff(s.poly_ptr)[:, None] * float(max(1, emax))
    tol = U.tolerance(s)
    assert np.abs((F[0] - Fw[0]).sum(1)).max() <= tol * size.max()
    assert (np.abs((J[0] - Jw[0, ..., :n]).sum(1)) <= 2 * tol * np.maximum(size, 1.0)).all()


@pytest.mark.parametrize("L,real", [(1, False), (2, False), (4, False), (4, True)])
@pytest.mark.parametrize("zeros", [1, 2, 5])
def test_zero_variables(pe, L, real, zeros):
    """Variables that are zero: monomials with one such factor of exponent 1, of exponent 2, with two."""
    n = 20
    s = ragged((41, L), L, n, [600, 37, 600, 0], 5, 2, real)
    x = points((42, L), 1, n, L, real)
    x[:, :, :, [3, 7, 8, 11, 19][:zeros]] = 0.0
    F, J = evaluate(pe, s, x, real)
    check(s, x[0], F[0], J[0], range(4))


@pytest.mark.parametrize("L,n,mons", [(2, 900, [300, 250]), (4, 600, [500, 300])])
def test_small_table(pe, L, n, mons):
    """The table of x alone with zero variables and with a variable out of range, and the adjoint."""
    import torch
    s = ragged((45, L), L, n, mons, 12, 3, False)
    x = points((46, L), 3, n, L, False)
    x[1, :, :, [3, 70, 71, 500]] = 0.0
    x[2, :, :, 9] *= 2.0**-310
    F, J = evaluate(pe, s, x, False)
    for pt in range(3):
        check(s, x[pt], F[pt], J[pt], range(len(mons)))
    v = synth.unit_circle_points(synth.rng_for((47, L)), 3, len(mons), L)
    S = pe.System.from_sparse(s)
    g = S.adjoint(U.to_device(x), U.to_device(v)).cpu().numpy()
    torch.cuda.synchronize()
    S.close()
    import oracle as O
    cols = [0, 3, 9, 71, n - 1]
    for pt in range(3):
        exact = O.adjoint_columns(s, x[pt], v[pt], cols)
        Sc = O.abs_sums_columns(s, x[pt], cols)
        av = np.hypot(v[pt, 0].sum(axis=0), v[pt, 1].sum(axis=0))
        for j in cols:
            scale = sum(q * av[p] for p, q in Sc[j].items())
            assert O.rel_error(g[pt, 0, :, j], g[pt, 1, :, j], exact[j], scale) <= 3 * U.tolerance(s)


@pytest.mark.parametrize("L,real", [(1, False), (2, False), (4, False), (4, True)])
@pytest.mark.parametrize("kind", ["range", "product", "zero"])
def test_points_out_of_range(pe, L, real, kind):
    """Factors beyond 2^300 whose products are in range ("range", and with a zero variable "zero"); factors within
    2^250 whose product is beyond 2^900 ("product"): every partial derivative as its own product."""
    n, m = 24, 600
    rng = synth.rng_for((51, L))
    two = lambda: np.stack([np.sort(rng.choice(12, size=2, replace=False)) for _ in range(3 * m)])  # noqa: E731
    var = np.concatenate([two(), 12 + two()], 1).astype(np.int32)
    lift = np.where(np.arange(n) < 12, 2.0**-310, 2.0**310)
    if kind == "product":  # in rows 0 and 1; row 2 stays in range
        lift = np.where(np.arange(n) < 12, 2.0**-240, 2.0**240)
        var[7] = [12, 13, 14, 15]
        var[m + 9] = [0, 1, 2, 3]
    s = synth.PolySystem(level=L, n_vars=n, poly_ptr=np.arange(0, 3 * m + 1, m, dtype=np.int64),
                         mon_ptr=np.arange(0, 12 * m + 1, 4, dtype=np.int64), var_idx=var.reshape(-1),
                         exps=np.ones(12 * m, np.int32), coef=synth.unit_circle(rng, 3 * m, L))
    if real:
        s.coef[1] = 0.0
    x = points((52, L), 1, n, L, real) * lift
    if kind == "zero":
        x[:, :, :, 5] = 0.0
    F, J = evaluate(pe, s, x, real)
    check(s, x[0], F[0], J[0], range(3))


@pytest.mark.parametrize("L,real", [(1, False), (2, False), (4, False), (2, True), (4, True)])
@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf, np.finfo(np.float64).max])
def test_nonfinite_points(pe, L, real, bad):
    """A NaN, an infinity or the largest double in one variable: entries are finite where the reverse sweep's are,
    and equal to it there."""
    n, wide = 30, 1200
    s = ragged((61, L), L, n, [400, 30, 700], 4, 1, real)
    x = points((62, L), 1, n, L, real)
    x[0, 0, :, 4] = 0.0
    x[0, 0, 0, 4] = bad
    F, J = evaluate(pe, s, x, real)
    Fw, Jw = evaluate(pe, widened(s, wide), np.concatenate([x, np.zeros((1, 2, L, wide - n))], 3), real)
    ok = lambda a: np.isfinite(a).all(axis=(1, 2))  # noqa: E731
    assert np.array_equal(ok(F), ok(Fw)) or np.isfinite(bad)
    fin = ok(J) & ok(Jw[..., :n])
    assert np.array_equal(ok(J), ok(Jw[..., :n])) or np.isfinite(bad)
    d = np.abs((J - Jw[..., :n]).sum(2)).max(axis=1)
    scale = np.maximum(1.0, np.abs(Jw[..., :n].sum(2)).max(axis=1))
    assert (d[fin] <= 1000 * U.tolerance(s) * scale[fin]).all()


@pytest.mark.parametrize("L", [1, 2, 4])
def test_adjoint_and_batch(pe, L):
    """J^H v from values, with a zero weight and a zero variable, against J; a batch with the bits of pe_eval."""
    import torch
    n, P = 48, 3
    s = ragged((71, L), L, n, [700, 64, 0, 701, 1], 6, 3, False)
    t = ragged((72, L), L, 20, [65] * 6, 5, 1, False)
    x, y = points((73, L), P, n, L, False), points((74, L), P, 20, L, False)
    x[1, :, :, 9] = 0.0
    v = synth.unit_circle_points(synth.rng_for((75, L)), P, 5, L)
    v[2, :, :, 3] = 0.0
    S, T = pe.System.from_sparse(s), pe.System.from_sparse(t)
    if T.info()["segment"] != S.info()["segment"]:
        T.set_shape(0, segment=S.info()["segment"])
    F, J = S.eval(U.to_device(x))
    F2, J2 = T.eval(U.to_device(y))
    g = S.adjoint(U.to_device(x), U.to_device(v)).cpu().numpy()
    B = pe.Batch([S, T])
    Fb, Jb = B.eval(torch.cat([U.to_device(x).reshape(-1), U.to_device(y).reshape(-1)]), P)
    torch.cuda.synchronize()
    assert torch.equal(Fb, torch.cat([F.reshape(-1), F2.reshape(-1)]))
    assert torch.equal(Jb, torch.cat([J.reshape(-1), J2.reshape(-1)]))
    J = J.cpu().numpy()
    import oracle as O
    tol = U.tolerance(s)
    for pt in range(P):
        Sc = O.abs_sums_columns(s, x[pt], range(n))
        av = np.hypot(v[pt, 0].sum(axis=0), v[pt, 1].sum(axis=0))
        V = [O.cdy_from_limbs(v[pt, 0, :, p], v[pt, 1, :, p]) for p in range(5)]
        for j in range(n):
            e = O.ZERO
            for p in range(5):
                e = O.cdy_add(e, O.cdy_mul(O.cdy_conj(O.cdy_from_limbs(J[pt, 0, :, p, j], J[pt, 1, :, p, j])), V[p]))
            scale = sum(q * av[p] for p, q in Sc[j].items())
            assert O.rel_error(g[pt, 0, :, j], g[pt, 1, :, j], e, scale) <= 3 * tol
    for h in (B, S, T):
        h.close()


def test_replay(pe):
    """A captured evaluation at points that change between the replays, zeros and out-of-range values among them."""
    import torch
    n, P = 40, 2
    s = ragged((81,), 2, n, [600, 100, 1025], 5, 2, False)
    S = pe.System.from_sparse(s)
    x = U.to_device(points((82,), P, n, 2, False))
    F, J = S.eval(x)
    st = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=st):
        S.eval(x, out=(F, J))
    for i in range(4):
        x.copy_(U.to_device(points((83, i), P, n, 2, False)))
        if i & 1:
            x[0, :, :, 3] = 0.0
        if i & 2:
            x[1, 0, 0, 5] = 2.0**320
            x[1, 0, 1, 5] = 0.0
        want = S.eval(x)
        F.zero_()
        J.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(F, want[0]) and torch.equal(J, want[1])
    S.close()
