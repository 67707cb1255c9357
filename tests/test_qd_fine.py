"""The finer quad-double products of the evaluation through monomial values: normwise error against exact rationals, no
larger than the plain products' and half of it on average; nonoverlapping limbs; zeros."""
import ctypes
import os
import subprocess
from fractions import Fraction

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
U4 = Fraction(1, 2 ** 212)


@pytest.fixture(scope="module")
def fine(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("qf") / "qd_fine.so")
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-shared", "-fPIC",
                    os.path.join(HERE, "qd_fine_host.cpp"), "-o", so], check=True)
    lib = ctypes.CDLL(so)

    def run(a):
        out = np.zeros_like(a)
        lib.pe_test_qd_fine(len(a), a.ctypes.data_as(ctypes.c_void_p), out.ctypes.data_as(ctypes.c_void_p))
        return out
    return run


def exact(limbs):
    return sum((Fraction(float(x)) for x in limbs), Fraction(0))


def operands(rng, count, cancel):
    """[count, 4, 4]: random quad doubles of widely different size; the second product near minus the first if `cancel`."""
    a = rng.uniform(0.5, 1.5, size=(count, 4, 4)) * rng.choice([-1.0, 1.0], size=(count, 4, 4))
    a *= 2.0 ** (-54.0 * np.arange(4))
    a *= 2.0 ** rng.integers(-40, 41, size=(count, 4, 1))
    if cancel:
        a[:, 2], a[:, 3] = -a[:, 0], a[:, 1]
        a[:, 3, 1:] *= 0.75
    return np.ascontiguousarray(a)


@pytest.mark.parametrize("cancel", [False, True])
def test_error(fine, cancel):
    a = operands(np.random.default_rng(7), 400, cancel)
    r = fine(a.reshape(-1, 16)).reshape(-1, 4, 4)
    err = np.zeros((len(a), 4))
    for i in range(len(a)):
        v = [exact(q) for q in a[i]]
        want = [v[0] * v[1]] * 2 + [v[0] * v[1] + v[2] * v[3]] * 2
        size = [abs(v[0] * v[1])] * 2 + [abs(v[0] * v[1]) + abs(v[2] * v[3])] * 2
        err[i] = [float(abs(exact(r[i, k]) - want[k]) / (size[k] * U4)) for k in range(4)]
    # 30 roundings of at most half a unit of order 4 at worst
    assert err[:, [0, 2]].max() <= 16
    assert err[:, 0].mean() <= 0.75 * err[:, 1].mean() and err[:, 2].mean() <= 0.75 * err[:, 3].mean()
    if not cancel:  # (where the sum of two products cancels, the plain one's limbs overlap too)
        lead = np.abs(r[:, :, :3])
        assert (np.abs(r[:, :, 1:]) <= 2.0 ** -51 * lead)[lead > 0].all()


def test_zeros(fine):
    a = operands(np.random.default_rng(8), 8, False)
    a[:4, 0] = 0.0
    a[2:4, 2] = 0.0
    r = fine(a.reshape(-1, 16)).reshape(-1, 4, 4)
    assert not r[:4, :2].any() and not r[2:4].any() and r[4:].any(axis=2).all()
