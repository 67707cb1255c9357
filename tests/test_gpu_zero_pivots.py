"""R and Q of a problem with a zero pivot in a later panel: what the panels before it gave, zeros from there on, and
nothing that was in the workspace."""
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


@pytest.mark.parametrize("L,real,n,at", [(1, False, 100, 70), (2, False, 100, 70), (4, False, 70, 40), (2, True, 140, 90),
                                         (2, False, 40, 3)])
def test_zero_pivot_in_a_panel(pe, L, real, n, at):
    import torch
    N, B = n + 9, 64 if real else 32
    rng = synth.rng_for((601, L, n))
    Ab = T._limbs((602, L, n), rng.standard_normal((2, 1 if real else 2, N, n + 1)), L)
    Ab[1, ..., at] = Ab[1, ..., 1]
    d = U.to_device(Ab)
    ws = torch.full(((pe._lib.pe_lstsq_workspace_bytes(L | (pe.PE_REAL if real else 0), 2, N, n) + 7) // 8,), 3.25,
                    dtype=torch.float64, device="cuda")
    x, resid, R, Q = pe.lstsq(d, want_R=True, want_Q=True, workspace=ws)
    torch.cuda.synchronize()
    x, resid, R, Q = [t.cpu().numpy() for t in (x, resid, R, Q)]
    assert resid[0, 1] > 0 and resid[1, 1] == -1.0 and not x[1].any()
    k0 = at // B * B
    assert not R[1][:, :, k0:].any() and not Q[1][..., k0:].any()
    if k0:
        lead = lambda a: a[0].sum(0) + (0 if real else 1j * a[1].sum(0))  # noqa: E731
        q, r, a = lead(Q[1])[:, :k0], lead(R[1])[:k0, :k0], lead(Ab[1])[:, :k0]
        assert np.abs(q @ r - a).max() <= 1e-12 and np.abs(q.conj().T @ q - np.eye(k0)).max() <= 1e-12
        assert np.abs(lead(R[1])[:k0, n] - q.conj().T @ lead(Ab[1])[:, n]).max() <= 1e-12 * N
