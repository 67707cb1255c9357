"""Columns with many slots in a chunk, which a wavefront adds together (eval_kernels.hpp, long_columns): lengths around
the line between the two orders, one to three long columns among 64, chunks in sequence, every kernel that owns columns."""
import numpy as np
import pytest

import gpu_util as U
import oracle as O
from paper_1402_2626_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pe():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_1402_2626_amd import polyeval
    return polyeval


def system(level, n, rows, real):
    """Row p has, for every (variable a, count m) of rows[p], m monomials c x_a x_b with b running over the others."""
    rng = synth.rng_for((91, n, level))
    var, ptr = [], [0]
    for row in rows:
        for a, m in row:
            others = [b for b in range(n) if b != a]
            var += [sorted((a, others[(7 * i) % len(others)])) for i in range(m)]
        ptr.append(len(var))
    coef = synth.unit_circle(rng, len(var), level)
    if real:
        coef[1] = 0.0
    return synth.PolySystem(level=level, n_vars=n, poly_ptr=np.array(ptr, np.int64),
                            mon_ptr=np.arange(0, 2 * len(var) + 1, 2, dtype=np.int64),
                            var_idx=np.array(var, np.int32).reshape(-1),
                            exps=rng.integers(1, 3, size=2 * len(var)).astype(np.int32), coef=coef)


WIDE = [[(5, 47)], [(5, 48)], [(63, 49)], [(64, 256)], [(129, 700)], [(5, 90), (6, 90)], [(5, 70), (6, 70), (7, 70)],
        [(0, 100), (127, 100)], []]
NARROW = [[(0, 47)], [(0, 48)], [(59, 60)], [(3, 30), (4, 30)]]


@pytest.mark.parametrize("L,real", [(1, False), (2, False), (4, False), (1, True), (2, True), (4, True)])
@pytest.mark.parametrize("n,rows", [(130, WIDE), (60, NARROW), (600, WIDE)])
def test_long_columns(pe, L, real, n, rows):
    import torch
    s = system(L, n, rows, real)
    P = 2
    x = synth.unit_circle_points(synth.rng_for((92, n)), P, n, L)
    if real:
        x[:, 1] = 0.0
        S = pe.System(pe.PE_REAL | L, n, s.poly_ptr, s.mon_ptr, s.var_idx, s.exps, np.ascontiguousarray(s.coef[:1]))
    else:
        S = pe.System.from_sparse(s)
    xd = U.to_device(x[:, :1] if real else x)
    F, J = S.eval(xd)
    torch.cuda.synchronize()
    full = lambda t: np.concatenate([t, np.zeros_like(t)], 1) if real else t  # noqa: E731
    Fh, Jh = full(F.cpu().numpy()), full(J.cpu().numpy())
    tol = U.tolerance(s)
    for pt in range(P):
        eF, eJ = U.max_errors_rows(s, x[pt], Fh[pt], Jh[pt], range(len(rows)), parallel=False)
        assert eF <= tol and eJ <= tol, (eF, eJ, tol)
    if not real:
        B = pe.Batch([S])
        Fb, Jb = B.eval(xd.reshape(-1), P)
        G = B.info()["chunks_per_workgroup"]
        B.close()
        S.set_shape(G)
        F, J = S.eval(xd)
        assert torch.equal(Fb, F.reshape(-1)) and torch.equal(Jb, J.reshape(-1))
        v = synth.unit_circle_points(synth.rng_for((93, n)), P, len(rows), L)
        g = S.adjoint(xd, U.to_device(v)).cpu().numpy()
        cols = [0, 3, 5, 6, 59, n - 1]
        for pt in range(P):
            exact = O.adjoint_columns(s, x[pt], v[pt], cols)
            Sc = O.abs_sums_columns(s, x[pt], cols)
            av = np.hypot(v[pt, 0].sum(axis=0), v[pt, 1].sum(axis=0))
            for j in cols:
                scale = sum(q * av[p] for p, q in Sc[j].items())
                assert O.rel_error(g[pt, 0, :, j], g[pt, 1, :, j], exact[j], scale) <= tol
    S.close()
