"""Truncated SVD at the edges of its paths: the last rows of a 32-row block, one block pair and just more,
the row and column limits of the single-workgroup forms, the first matrices of the QR start, and the
steep spectra whose rotations differ most in size."""
import numpy as np
import pytest

import oracle
import synth
from gpu_common import ctx, to_dev

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -53

SHAPES = [(2, 2), (2, 3), (17, 64), (31, 33), (32, 32), (32, 64), (32, 65), (33, 33), (63, 64), (64, 65), (64, 1024),
          (64, 1025), (65, 65), (65, 200), (96, 97), (127, 130), (161, 129), (255, 256), (257, 256), (289, 300)]


@pytest.mark.parametrize("m,n", SHAPES)
@pytest.mark.parametrize("ratio", [0.0, 0.25])
def test_svd_path_edges(m, n, ratio):
    """Against the oracle's spectrum and by reconstruction and orthonormality.  Tolerances: a backward-stable SVD
    leaves max(m, n) roundings per entry, taken 64 times as elsewhere.  ratio > 0: columns scaled by
    exp(-ratio j), down to 1e-14 of the first."""
    A = synth.random_matrix(m, n, 300 + 3 * m + n)
    if ratio:
        A = A * np.exp(-np.minimum(ratio * np.arange(n), 32.0))[None, :]
    R = min(m, n)
    k = R
    S, U, Vt, spec, kk, sw, st = ctx().svd_truncate(to_dev(A), k)
    S, U, Vt = S.cpu().numpy(), U.cpu().numpy(), Vt.cpu().numpy()
    So = oracle.svd(A)[0]
    tol = 64 * max(m, n) * EPS
    assert st == 0 and kk == k
    assert np.all(np.diff(S) <= 0.0)
    assert np.abs(S - So).max() <= tol * So[0]
    assert np.abs((U * S) @ Vt - A).max() <= tol * So[0]
    assert np.abs(U.T @ U - np.eye(k)).max() <= tol
    assert np.abs(Vt @ Vt.T - np.eye(k)).max() <= tol


@pytest.mark.parametrize("m,n", [(256, 256), (513, 511), (544, 520), (1023, 1030), (1060, 1057)])
def test_svd_qr_start_edges(m, n):
    """The QR start's panel forms (one workgroup of up to 8 or 16 waves, more than 1024 rows) and the last
    columns of its blocked products, alone and as a batch with the same numbers; tolerances as above."""
    As = np.stack([synth.random_matrix(m, n, 900 + m + 7 * i) for i in range(2)])
    k = min(m, n) // 2
    c = ctx()
    S, U, Vt, spec, sw, st = c.svd_truncate_batched(to_dev(As), k)
    assert st == 0
    tol = 64 * max(m, n) * EPS
    for i in range(2):
        s, u, v = S[i].cpu().numpy(), U[i].cpu().numpy(), Vt[i].cpu().numpy()
        ref = np.linalg.svd(As[i], compute_uv=False)
        assert np.abs(s - ref).max() <= tol * ref[0]
        assert np.abs(u.T @ u - np.eye(k)).max() <= tol
        assert np.abs(v @ v.T - np.eye(k)).max() <= tol
        assert np.abs(u.T @ As[i] - s[:k, None] * v).max() <= tol * ref[0]
        s1 = c.svd_truncate(to_dev(As[i]), k)[0].cpu().numpy()
        assert np.abs(s1 - s).max() <= tol * ref[0]
