"""Truncated SVD of matrices far from norm 1, and of matrices whose rows or columns run over ninety decades: the
squares of squared row norms leave the range of FP64 there, the factors must not notice.  Every path: at most
32 rows, one block pair, blocks without and with the QR start."""
import numpy as np
import pytest

import oracle
import synth
from gpu_common import ctx, to_dev

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -53

SHAPES = [(12, 15), (24, 40), (40, 64), (130, 64), (100, 120), (300, 280)]


def _svd(A):
    k = min(A.shape)
    S, U, Vt, spec, kk, sw, st = ctx().svd_truncate(to_dev(A), k)
    assert st == 0 and kk == k
    return S.cpu().numpy(), U.cpu().numpy(), Vt.cpu().numpy(), spec.cpu().numpy()


@pytest.mark.parametrize("m,n", SHAPES)
@pytest.mark.parametrize("e", [-460, -300, -270, -262, -255, 250, 256, 300, 460])
def test_scaled_by_a_power_of_two(m, n, e):
    """A 2^e against the oracle's SVD of A; tolerances as at norm 1 (max(m, n) roundings per entry, 64 times)."""
    A = synth.random_matrix(m, n, 40 + 3 * m + n)
    S, U, Vt, spec = _svd(np.ldexp(A, e))
    S = np.ldexp(S, -e)
    ref = oracle.svd(A)[0]
    tol = 64 * max(m, n) * EPS
    k = min(m, n)
    assert np.abs(S - ref).max() <= tol * ref[0]
    assert np.abs((U * S) @ Vt - A).max() <= tol * ref[0]
    assert np.abs(U.T @ U - np.eye(k)).max() <= tol
    assert np.abs(Vt @ Vt.T - np.eye(k)).max() <= tol
    p = ref ** 2 / (ref ** 2).sum()
    assert abs(spec[1] + (p * np.log(p)).sum()) <= tol


@pytest.mark.parametrize("m,n", [(320, 300), (300, 320)])
@pytest.mark.parametrize("side", [0, 1])
def test_graded_over_ninety_decades(m, n, side):
    """Rows (side 0) or columns scaled by 10^(-0.3 j): with the QR start every row is orthogonalised however short,
    so both factors stay orthonormal.  Tolerances as above."""
    d = 10.0 ** (-0.3 * np.arange((m, n)[side]))
    A = synth.random_matrix(m, n, 77) * (d[:, None] if side == 0 else d[None, :])
    S, U, Vt, spec = _svd(A)
    ref = np.linalg.svd(A, compute_uv=False)
    tol = 64 * max(m, n) * EPS
    k = min(m, n)
    assert np.abs(S - ref).max() <= tol * ref[0]
    assert np.abs((U * S) @ Vt - A).max() <= tol * ref[0]
    assert np.abs(U.T @ U - np.eye(k)).max() <= tol
    assert np.abs(Vt @ Vt.T - np.eye(k)).max() <= tol
