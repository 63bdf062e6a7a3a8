"""The host eigensolver of the Lanczos recurrence (CPU): lowest eigenpair of symmetric tridiagonals against a
dense eigensolver, whatever starting value it is given, and the residual estimate that screens records."""
import ctypes as C
import math

import numpy as np
import pytest

import paper_2604_03960_amd as tna

_dp = C.POINTER(C.c_double)
_low = getattr(tna._lib, "_ZN3tna19tridiag_lowest_hostEiPKdS1_Pdd")
_low.restype, _low.argtypes = C.c_double, [C.c_int, _dp, _dp, _dp, C.c_double]
_est = getattr(tna._lib, "_ZN3tna16tridiag_estimateEiPKdS1_dPdS2_")
_est.restype, _est.argtypes = C.c_bool, [C.c_int, _dp, _dp, C.c_double, _dp, _dp]


def _p(x):
    return x.ctypes.data_as(_dp)


def _matrices(n):
    rng = np.random.default_rng(n)
    for scale, off in ((1.0, 1.0), (1e-8, 1e-12), (50.0, 1e-3), (1.0, 10.0)):
        yield rng.standard_normal(n) * scale, np.abs(rng.standard_normal(n)) * off
    yield np.full(n, -3.0), np.abs(rng.standard_normal(n))  # an exactly zero first pivot at the diagonal
    b = np.abs(rng.standard_normal(n))
    b[n // 2] = 0.0
    yield rng.standard_normal(n), b  # decoupled blocks
    yield -4.0 + np.cumsum(rng.random(n)), np.exp(-0.7 * np.arange(n))  # a converging recurrence
    yield np.zeros(n), np.zeros(n)


@pytest.mark.parametrize("n", [1, 2, 3, 9, 33, 120])
def test_lowest_pair_from_any_start(n):
    """Eigenvalue to 16 roundings of the matrix norm per row of the pivot sequence, residual likewise."""
    for a, b in _matrices(n):
        T = np.diag(a) + np.diag(b[:n - 1], 1) + np.diag(b[:n - 1], -1)
        ex = np.linalg.eigvalsh(T)[0]
        tol = 16 * n * 2.0 ** -53 * max(np.abs(a).max() + 2 * np.abs(b).max(), 1e-300)
        for x0 in (math.nan, ex, ex + 1e-7, a.min(), 1e6, -1e6):
            y = np.zeros(n)
            lam = _low(n, _p(a), _p(b), _p(y), x0)
            assert abs(lam - ex) <= tol
            assert abs(np.linalg.norm(y) - 1.0) <= 1e-14
            assert np.linalg.norm(T @ y - lam * y) <= 4 * tol


def test_residual_estimate_screens_unconverged_records():
    """On a Lanczos recurrence the estimate agrees with the eigenvector's residual while that is large."""
    rng = np.random.default_rng(7)
    H = rng.standard_normal((150, 150))
    H = H + H.T - 40.0 * np.outer(*(2 * [np.eye(150)[0]]))
    V, al, be = [np.ones(150) / math.sqrt(150.0)], [], []
    for j in range(25):
        w = H @ V[j]
        al.append(V[j] @ w)
        for _ in range(2):
            for u in V:
                w = w - (u @ w) * u
        be.append(np.linalg.norm(w))
        V.append(w / be[-1])
    al, be = np.array(al), np.array(be)
    th, rr = al[0], be[0]
    seen = 0
    for n in range(2, 25):
        d = 0.5 * (al[n - 1] - th)
        x0 = 0.5 * (th + al[n - 1]) - math.hypot(d, rr)
        y = np.zeros(n)
        lam = _low(n, _p(al), _p(be), _p(y), math.nan)
        res = abs(be[n - 1] * y[n - 1])
        t, r = C.c_double(), C.c_double()
        if res > 1e-6 and _est(n, _p(al), _p(be), x0, C.byref(t), C.byref(r)):
            seen += 1
            assert abs(t.value - lam) <= 1e-12 * abs(lam)
            assert abs(r.value - res) <= 1e-2 * res
        th, rr = lam, res
    assert seen >= 5
