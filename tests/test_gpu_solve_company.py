"""A problem of the least-squares solver has the same bits whatever else a call holds: alone, among copies of itself,
in a trailing group, beside other systems of a batch."""
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


@pytest.mark.parametrize("L,real,N,n,P", [(1, False, 300, 40, 300), (2, False, 130, 70, 130), (2, True, 1100, 65, 40),
                                          (4, False, 200, 33, 20), (2, False, 20, 6, 40)])
def test_alone_and_among_others(pe, L, real, N, n, P):
    import torch
    rng = synth.rng_for((301, L, N))
    lead = rng.standard_normal((2, 1 if real else 2, N, n + 1))
    Ab = np.ascontiguousarray(np.moveaxis(synth.lower_limbs(rng, lead, L), 0, 2))
    two = U.to_device(Ab)
    many = two.repeat_interleave((P + 1) // 2, 0)[:P].contiguous()
    alone = [pe.lstsq(two[i:i + 1].contiguous(), want_R=True, want_Q=True) for i in range(2)]
    got = pe.lstsq(many, want_R=True, want_Q=True)
    torch.cuda.synchronize()
    for t in range(4):
        for p in range(P):
            assert torch.equal(got[t][p], alone[p // ((P + 1) // 2)][t][0]), (t, p)


@pytest.mark.parametrize("L", [1, 2])
def test_groups_of_a_call(pe, L):
    """More problems than 1 GiB of workspace holds at once: the last group is a small one."""
    import torch
    N, n, P = 70, 33, {1: 2700, 2: 1750}[L]
    rng = synth.rng_for((302, L))
    Ab = U.to_device(np.ascontiguousarray(np.moveaxis(synth.lower_limbs(rng, rng.standard_normal((1, 2, N, n + 1)), L), 0, 2)))
    nbytes = [pe._lib.pe_lstsq_workspace_bytes(L, p, N, n) for p in (1, P)]
    assert nbytes[1] < P * nbytes[0] and nbytes[1] // nbytes[0] < P
    one = pe.lstsq(Ab)[0]
    x = pe.lstsq(Ab.expand(P, -1, -1, -1, -1).contiguous())[0]
    torch.cuda.synchronize()
    assert torch.equal(x, one.expand(P, -1, -1, -1))


@pytest.mark.parametrize("L", [1, 2, 4])
def test_newton_points_and_batch(pe, L):
    """A Newton step of one point, of many, and of the system in a batch."""
    import torch
    sizes, P = [(90, 70), (150, 140), (40, 33)], 24
    systems = [synth.random_system((303, L, N), L, n_vars=n, n_polys=N, m=12, k=4) for N, n in sizes]
    S = [pe.System.from_sparse(s) for s in systems]
    for t in S[1:]:
        if t.info()["segment"] != S[0].info()["segment"]:
            t.set_shape(0, segment=S[0].info()["segment"])
    xs = [U.to_device(synth.unit_circle_points(synth.rng_for((304, n)), P, n, L)) for _, n in sizes]
    B = pe.Batch(S)
    xb, _ = B.newton_step(torch.cat([x.reshape(-1) for x in xs]), P)
    at = 0
    for T, x in zip(S, xs):
        y, _ = T.newton_step(x.clone())
        z, _ = T.newton_step(x[5:6].clone())
        torch.cuda.synchronize()
        assert torch.equal(y[5:6], z)
        assert torch.equal(xb[at:at + x.numel()], y.reshape(-1))
        at += x.numel()
    for h in [B] + S:
        h.close()
