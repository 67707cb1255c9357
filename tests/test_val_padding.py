"""The value layout's packer refuses systems whose column lists would be mostly padding, and no others."""
import ctypes

import numpy as np
import pytest

from paper_1402_2626_amd import synth
from test_val_packer import lib  # noqa: F401  (the packer built for the host)


def pack(lib, s, block_mons=65534):  # noqa: F811
    sz = np.zeros(13, np.int64)
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)  # noqa: E731
    arr = [np.ascontiguousarray(a, t) for a, t in ((s.poly_ptr, np.int64), (s.mon_ptr, np.int64),
                                                   (s.var_idx, np.int32), (s.exps, np.int32))]
    ok = lib.pe_test_val_pack(s.n_vars, s.n_polys, *[p(a) for a in arr], block_mons, p(sz))
    return ok, int(sz[6])


def common(n, N, m, k, long):
    """Every monomial holds the variables 0 .. long - 1 and k - long others."""
    rng = synth.rng_for((411, n, long))
    rest = long + synth.distinct_sorted_subsets(rng, N * m, n - long, k - long)
    var = np.concatenate([np.tile(np.arange(long), (N * m, 1)), rest], 1).astype(np.int32)
    return synth.PolySystem(level=1, n_vars=n, poly_ptr=np.arange(0, N * m + 1, m, dtype=np.int64),
                            mon_ptr=np.arange(0, N * m * k + 1, k, dtype=np.int64), var_idx=var.reshape(-1),
                            exps=np.ones(N * m * k, np.int32), coef=np.ones((2, 1, N * m)))


@pytest.mark.parametrize("n,N,m,k,long,ok", [
    (512, 40, 1500, 5, 1, 0),    # one long column among 512: 64 / 5 entries per occurrence
    (512, 40, 1500, 5, 0, 1),    # the same without it
    (512, 2, 1500, 5, 1, 1),     # below 1 MB: taken
    (64, 40, 1500, 8, 1, 1),     # eight lanes per column: 64 / 8 / 8 and the short ones
    (512, 20, 1500, 40, 24, 1),  # many long columns fill their slices
])
def test_padding(lib, n, N, m, k, long, ok):  # noqa: F811
    s = common(n, N, m, k, long)
    got, entries = pack(lib, s)
    assert got == ok
    if ok:
        assert entries <= 4 * s.nnz + (1 << 18)
