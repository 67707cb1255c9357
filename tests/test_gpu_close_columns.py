"""Panels that plain modified Gram-Schmidt takes (bl_mgs_panel): every panel or one, fewer and more workgroups than
columns, several problems at once, columns close enough to be taken twice, chains of such columns, a zero pivot on the
way, replays from a graph."""
import numpy as np
import pytest

import gpu_util as U
import test_gpu_blockls as T
from paper_1402_2626_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pe():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_1402_2626_amd import polyeval
    return polyeval


def close(seed, P, C, N, n, eps, B, chain):
    """In every panel of B columns, columns that agree to eps with the panel's first, or each with the one before it."""
    rng = synth.rng_for(seed)
    a = rng.standard_normal((P, C, N, n + 1))
    for k0 in range(0, n, B):
        for j in range(k0 + 1, min(n, k0 + B)):
            a[..., j] = a[..., j - 1 if chain and j % 3 else k0] + eps * a[..., j]
    return a


@pytest.mark.parametrize("L,real,N,n,eps,chain", [
    (1, False, 70, 40, 1e-5, False), (1, True, 300, 66, 1e-6, False), (2, False, 50, 33, 1e-8, False),
    (2, False, 700, 70, 1e-9, True), (2, False, 300, 64, 1e-13, False), (2, True, 1100, 130, 1e-8, True),
    (4, False, 90, 35, 1e-10, False), (4, True, 300, 70, 1e-15, True)])
def test_close_columns(pe, L, real, N, n, eps, chain):
    rng = synth.rng_for((701, L, N))
    Ab = T._limbs((702, L, N), close((703, L, N), 3, 1 if real else 2, N, n, eps, 64 if real else 32, chain), L)
    x, resid, R, Q = T._solve(pe, Ab)
    assert (resid[:, 1] > 0).all()
    for p in (0, 2):
        T._check(Ab[p], x[p], R[p], Q[p], L, rng, count=8)


@pytest.mark.parametrize("L", [1, 2])
def test_zero_pivot_and_replay(pe, L):
    """A zero pivot among close columns ends that problem only; the same bits from a graph, which is captured before
    the matrices are there."""
    import torch
    N, n, P = 200, 70, 4
    Ab = T._limbs((711, L), close((712, L), P, 2, N, n, 1e-6, 32, False), L)
    Ab[1, ..., 40] = Ab[1, ..., 33]
    Ab[2, ..., 5] = Ab[2, ..., 3]
    d = U.to_device(Ab)
    want = pe.lstsq(d)
    torch.cuda.synchronize()
    r = want[1].cpu().numpy()
    assert r[0, 1] > 0 and r[3, 1] > 0 and r[1, 1] == -1.0 and r[2, 1] == -1.0
    for p in (0, 3):
        assert torch.equal(pe.lstsq(d[p:p + 1].contiguous())[0][0], want[0][p])
    nbytes = pe._lib.pe_lstsq_workspace_bytes(L, P, N, n)
    ws = torch.empty((nbytes + 7) // 8, dtype=torch.float64, device="cuda")
    buf = torch.zeros_like(d)
    st = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=st):
        got = pe.lstsq(buf, workspace=ws)
    for i in range(3):
        buf.copy_(d if i != 1 else d.flip(0))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(got[0] if i != 1 else got[0].flip(0), want[0])
