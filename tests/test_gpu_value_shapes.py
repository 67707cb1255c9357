"""The launch shape of a system evaluated through monomial values: it changes neither the algorithm nor the bits, and
tuning keeps it."""
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


def system(level, real):
    """Rows of 200 monomials of 16 variables: two chunks at segment 8, one at segment 16 (double)."""
    s = synth.random_system((401, level), level, n_vars=64, n_polys=24, m=200, k=16)
    if real:
        s.coef[1] = 0.0
    return s


@pytest.mark.parametrize("L,real,segments", [(1, False, (8, 16)), (1, True, (8, 16)), (2, True, (8, 6, 4)),
                                             (2, False, (8, 6, 4)), (4, False, (4, 2))])
def test_shape_keeps_the_bits(pe, L, real, segments):
    import torch
    s = system(L, real)
    x = synth.unit_circle_points(synth.rng_for((402, L)), 2, 64, L)
    if real:
        S = pe.System(pe.PE_REAL | L, 64, s.poly_ptr, s.mon_ptr, s.var_idx, s.exps, np.ascontiguousarray(s.coef[:1]))
        x = np.where(np.abs(x[:, :1]) < 0.3, 0.75, x[:, :1])
        x[:, :, 1:] = 0.0
    else:
        S = pe.System.from_sparse(s)
    xd = U.to_device(x)
    v = U.to_device(synth.unit_circle_points(synth.rng_for((403, L)), 2, 24, L))
    assert S.info()["segment"] == segments[0]
    F, J = S.eval(xd)
    g = None if real else S.adjoint(xd, v)
    for seg in segments[1:] + segments[:1]:
        S.set_shape(0, segment=seg)
        F1, J1 = S.eval(xd)
        torch.cuda.synchronize()
        assert torch.equal(F, F1) and torch.equal(J, J1), seg
        assert real or torch.equal(g, S.adjoint(xd, v)), seg
        V, G = S.eval_terms(xd)
        torch.cuda.synchronize()
        assert np.allclose(V.cpu().numpy()[:, 0, 0].reshape(2, 24, 200).sum(2), F.cpu().numpy()[:, 0, 0], rtol=0, atol=1e-10)
    S.close()


def test_tuning_keeps_the_shape(pe, tmp_path):
    """Systems of one batch stay in step when they are tuned, whatever the clock says."""
    S = [pe.System.from_sparse(synth.random_system((404, m), 2, n_vars=64, n_polys=24, m=m, k=16)) for m in (100, 150, 200)]
    cache = tmp_path / "plans.txt"
    pe.set_plan_cache(str(cache))
    try:
        for t in S:
            t.set_shape(0, segment=6)
            before = t.info()
            t.autotune(P=2)
            after = t.info()
            assert (after["segment"], after["chunks_per_workgroup"]) == (6, before["chunks_per_workgroup"])
        assert all("| 6 " in line for line in cache.read_text().strip().splitlines())
        pe.Batch(S).close()
    finally:
        pe.set_plan_cache(None)
    for t in S:
        t.close()
