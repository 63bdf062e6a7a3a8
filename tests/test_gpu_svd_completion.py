"""Kept null vectors of rank-deficient matrices: their completion leaves both factors orthonormal also where the
complement has so few dimensions that no unit vector lies mostly in it."""
import numpy as np
import pytest

import synth
from gpu_common import ctx, to_dev

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -53


@pytest.mark.parametrize("m,n", [(2, 2), (16, 16), (16, 17), (32, 64), (64, 64), (60, 130), (128, 128), (256, 256),
                                 (257, 258), (300, 257)])
@pytest.mark.parametrize("side", [0, 1])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_full_rank_kept_of_a_deficient_matrix(m, n, side, dtype):
    """Every third row or second column zero.  Tolerances: max(m, n) roundings of the type, 64 times."""
    import torch
    A = synth.random_matrix(m, n, 11 + m + n)
    if side == 0:
        A[::3] = 0.0
    else:
        A[:, ::2] = 0.0
    A = A.astype(dtype)
    k = min(m, n)
    S, U, Vt, spec, kk, sw, st = ctx().svd_truncate(torch.from_numpy(A).cuda(), k)
    S, U, Vt = S.cpu().numpy(), U.cpu().numpy().astype(float), Vt.cpu().numpy().astype(float)
    ref = np.linalg.svd(A.astype(float), compute_uv=False)
    tol = 64 * max(m, n) * (EPS if dtype == np.float64 else 2.0 ** -24)
    assert st == 0 and kk == k
    assert np.abs(S - ref).max() <= tol * ref[0]
    assert np.abs((U * S) @ Vt - A).max() <= tol * ref[0]
    assert np.abs(U.T @ U - np.eye(k)).max() <= tol
    assert np.abs(Vt @ Vt.T - np.eye(k)).max() <= tol
