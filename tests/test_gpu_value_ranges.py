"""Evaluation through monomial values (value_kernels.hpp) where a value or a partial product leaves the range in which
the division by x_v is exact enough: F beside zero and out-of-range variables, coefficients and weights that are tiny or
not finite, products that leave the range and come back.  Against the exact oracle with the tolerance of the other
evaluation tests, and for what is finite against the reverse sweep (the same monomials over more variables)."""
import numpy as np
import pytest

import gpu_util as U
import oracle as O
import test_gpu_values as V
from paper_1402_2626_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pe():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_1402_2626_amd import polyeval
    return polyeval


def uniform(seed, level, n, N, m, pick, coef=None):
    """N polynomials of m monomials over the variables pick(rng, p, i), exponents 1."""
    rng = synth.rng_for(seed)
    var = [np.sort(np.asarray(pick(rng, p, i), np.int32)) for p in range(N) for i in range(m)]
    k = np.array([len(v) for v in var])
    return synth.PolySystem(level=level, n_vars=n, poly_ptr=np.arange(0, N * m + 1, m, dtype=np.int64),
                            mon_ptr=np.concatenate([[0], np.cumsum(k)]).astype(np.int64), var_idx=np.concatenate(var),
                            exps=np.ones(int(k.sum()), np.int32),
                            coef=synth.unit_circle(rng, N * m, level) if coef is None else coef)


def sweep(pe, s, x, wide):
    """F and J of the reverse sweep."""
    F, J = V.evaluate(pe, V.widened(s, wide), np.concatenate([x, np.zeros(x.shape[:3] + (wide - s.n_vars,))], 3), False)
    return F, J[..., :s.n_vars]


# the table of x alone (emax 4 at these n) and the full table
@pytest.mark.parametrize("L,n,emax", [(2, 900, 4), (4, 600, 3), (1, 40, 2), (2, 40, 2), (4, 40, 2)])
def test_zero_beside_out_of_range(pe, L, n, emax):
    """Exact zeros and a variable out of range at one point: F with J, F alone and in a batch."""
    import torch
    s = V.ragged((201, L, n), L, n, [700, 690], 10, emax, False)
    x = V.points((202, L), 2, n, L, False)
    x[:, :, :, [3, 7, n // 2]] = 0.0
    x[0, :, :, 9] *= 2.0**-310
    x[1, :, :, 11] *= 2.0**(310 if emax < 4 else 240)  # beyond 2^(900 / emax); its powers are representable
    F, J = V.evaluate(pe, s, x, False)
    F1, _ = V.evaluate(pe, s, x, False, want_J=False)
    assert np.array_equal(F, F1)
    for pt in range(2):
        V.check(s, x[pt], F[pt], J[pt], range(2))
    S = pe.System.from_sparse(s)
    B = pe.Batch([S])
    Fb, Jb = B.eval(U.to_device(x).reshape(-1), 2)
    torch.cuda.synchronize()
    assert np.array_equal(Fb.cpu().numpy(), F.reshape(-1)) and np.array_equal(Jb.cpu().numpy(), J.reshape(-1))
    B.close()
    S.close()


@pytest.mark.parametrize("L,n", [(2, 900), (4, 600), (2, 40)])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_zero_times_nonfinite(pe, L, n, bad):
    """A variable that is not finite and occurs beside a zero only: F is not finite where the sweep's is not."""
    others = np.array([v for v in range(n) if v not in (3, 9)])

    def pick(rng, p, i):
        if p == 0 and i == 5:
            return [3, 9] + list(rng.choice(others, size=8, replace=False))
        return rng.choice(others, size=10, replace=False)

    s = uniform((211, L), L, n, 2, 400, pick)
    s.exps[::7] = 4
    x = V.points((212, L), 1, n, L, False)
    x[0, :, :, 3] = 0.0
    x[0, :, :, 9] = 0.0
    x[0, 0, 0, 9] = bad
    F, J = V.evaluate(pe, s, x, False)
    Fw, Jw = sweep(pe, s, x, 4 * n + s.nnz // 2)
    ok = lambda a: np.isfinite(a).all(axis=(1, 2))  # noqa: E731
    assert np.array_equal(ok(F), ok(Fw)) and not ok(F)[0, 0] and ok(F)[0, 1]
    assert np.array_equal(ok(J), ok(Jw))


# |x|, |coefficient|, as powers of two: the product of four variables is in range, the value is not
TINY = [(1, -180, -350), (2, -180, -350), (4, -170, -250)]


@pytest.mark.parametrize("L,ex,ec", TINY)
def test_tiny_coefficients(pe, L, ex, ec):
    """Values that underflow where the derivatives are normal numbers; rows 1 and 2 hold one such monomial and none.
    J only: the terms of F themselves are not representable."""
    n, m = 24, 600
    s = uniform((221, L), L, n, 3, m, lambda rng, p, i: rng.choice(12, size=4, replace=False) + 12 * (i & 1))
    s.coef[:, :, :m] *= 2.0**ec
    s.coef[:, :, m + 8] *= 2.0**ec
    x = V.points((222, L), 1, n, L, False)
    x[:, :, :, :12] *= 2.0**ex
    s.coef[:, :, 1:m:2] *= 2.0**(4 * ex - ec)  # the odd monomials of row 0 are as small, by their coefficients
    _, J = V.evaluate(pe, s, x, False)
    _, eJ = U.max_errors_rows(s, x[0], np.zeros_like(J[0, :, :, :, 0]), J[0], range(3), parallel=False)
    assert eJ <= U.tolerance(s), (eJ, U.tolerance(s))


def check_adjoint(s, x, v, g, cols):
    exact = O.adjoint_columns(s, x, v, cols)
    Sc = O.abs_sums_columns(s, x, cols)
    av = np.hypot(v[0].sum(axis=0), v[1].sum(axis=0))
    for j in cols:
        scale = sum(q * av[p] for p, q in Sc[j].items())
        assert O.rel_error(g[0, :, j], g[1, :, j], exact[j], scale) <= 3 * U.tolerance(s), j


@pytest.mark.parametrize("L,ex,ev", TINY)
def test_tiny_weights(pe, L, ex, ev):
    """The same through the adjoint's weights."""
    import torch
    n, m = 24, 600
    s = uniform((231, L), L, n, 3, m, lambda rng, p, i: rng.choice(12, size=4, replace=False) + 12 * (p == 2))
    x = V.points((232, L), 1, n, L, False)
    x[:, :, :, :12] *= 2.0**ex
    v = synth.unit_circle_points(synth.rng_for((233, L)), 1, 3, L)
    v[..., :2] *= 2.0**ev
    S = pe.System.from_sparse(s)
    g = S.adjoint(U.to_device(x), U.to_device(v)).cpu().numpy()
    torch.cuda.synchronize()
    S.close()
    check_adjoint(s, x[0], v[0], g[0], [0, 5, 11, 12, 23])


@pytest.mark.parametrize("L", [1, 2, 4])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_nonfinite_weight(pe, L, bad):
    """A weight that is not finite reaches the variables of its polynomial and no others."""
    import torch
    n, m = 40, 600
    s = uniform((241, L), L, n, 4, m, lambda rng, p, i: rng.choice(20, size=4, replace=False) + 20 * (p & 1))
    x = V.points((242, L), 1, n, L, False)
    v = synth.unit_circle_points(synth.rng_for((243, L)), 1, 4, L)
    v[0, 0, 0, 2] = bad
    S = pe.System.from_sparse(s)
    g = S.adjoint(U.to_device(x), U.to_device(v)).cpu().numpy()[0]
    torch.cuda.synchronize()
    S.close()
    assert not np.isfinite(g[:, :, :20]).all(axis=(0, 1)).any()
    assert np.isfinite(g[:, :, 20:]).all()
    v[0, :, :, 2] = 0.0
    check_adjoint(s, x[0], v[0], g, [20, 31, 39])


@pytest.mark.parametrize("L", [1, 2, 4])
@pytest.mark.parametrize("lanes", [1, 2])
def test_partial_products_out_of_range(pe, L, lanes):
    """Factors whose product is near 1 while the product of a lane's first four, or of all a lane has, is near 2^-1000."""
    n, m = 24, 600
    if lanes == 1:
        pick = lambda rng, p, i: np.concatenate([rng.choice(12, 4, replace=False), 12 + rng.choice(12, 4, replace=False)])  # noqa: E731
        lift = np.where(np.arange(n) < 12, 2.0**-250, 2.0**250)
    else:
        pick = lambda rng, p, i: np.arange(n)  # noqa: E731
        lift = np.where(np.arange(n) % 2 == 0, 2.0**-83, 2.0**83)
    s = uniform((251, L), L, n, 3, m, pick)
    x = V.points((252, L), 1, n, L, False) * lift
    F, J = V.evaluate(pe, s, x, False)
    V.check(s, x[0], F[0], J[0], range(3))


@pytest.mark.parametrize("L", [1, 2, 4])
@pytest.mark.parametrize("lift", [0, 1, 3])
def test_long_products(pe, L, lift):
    """Products of 600 variables (quad double, which takes fewer: 200) of modulus 1 or by halves 2^-lift and 2^lift
    (2^-3lift, 2^3lift): on the way they reach 2^(-300 lift)."""
    n, m = 600 if L < 4 else 200, 2
    lift *= 600 // n
    s = uniform((261, L), L, n, 1, m, lambda rng, p, i: np.arange(n))
    x = V.points((262, L, lift), 1, n, L, False) * np.where(np.arange(n) < n // 2, 2.0**-lift, 2.0**lift)
    F, J = V.evaluate(pe, s, x, False)
    V.check(s, x[0], F[0], J[0], range(1))
