"""Truncated SVD with the QR start (at least 256 rows) of matrices whose rows or columns run down to where their
squares underflow, and of matrices whose columns are all the same: no reflector of such a column may leave the range
of FP64, and no index may follow from a value that does."""
import numpy as np
import pytest

import synth
from gpu_common import ctx, to_dev

pytestmark = pytest.mark.gpu
EPS = 2.0 ** -53


def _check(A, k):
    S, U, Vt, spec, kk, sw, st = ctx().svd_truncate(to_dev(A), k)
    S, U, Vt = S.cpu().numpy(), U.cpu().numpy(), Vt.cpu().numpy()
    ref = np.linalg.svd(A, compute_uv=False)
    tol = 64 * max(A.shape) * EPS  # as for the other shapes
    assert st == 0 and kk == k
    assert np.abs(S - ref).max() <= tol * ref[0]
    assert np.abs(U.T @ A - S[:k, None] * Vt).max() <= tol * ref[0]
    assert np.abs(U.T @ U - np.eye(k)).max() <= tol
    assert np.abs(Vt @ Vt.T - np.eye(k)).max() <= tol


@pytest.mark.parametrize("panel", ["", "col", "coop"])
@pytest.mark.parametrize("m,n", [(256, 256), (257, 300), (300, 256)])
@pytest.mark.parametrize("side", [0, 1])
@pytest.mark.parametrize("decades", [166, 290])
def test_graded_into_underflow(m, n, side, decades, panel, monkeypatch):
    if panel:
        monkeypatch.setenv("TNA_QR_PANEL", panel)
    L = (m, n)[side]
    d = 10.0 ** (-decades * np.arange(L) / (min(m, n) - 1.0)).clip(1e-300)
    _check(synth.random_matrix(m, n, 7 + m) * (d[:, None] if side == 0 else d[None, :]), min(m, n) // 2)


@pytest.mark.parametrize("m,n", [(256, 256), (257, 300), (1040, 1030)])
def test_equal_columns_and_rank_one(m, n):
    x, y = synth.random_matrix(m, 1, 3), synth.random_matrix(1, n, 4)
    _check(np.tile(x, (1, n)), 3)
    _check(np.tile(y, (m, 1)), 3)
    _check(x @ y, 3)


def test_equal_rows_left_far_below_the_norm():
    """300 equal entries in each of 257 columns: the QR start leaves some 200 equal rows at 1e-92 of the norm with 43
    columns between them."""
    _check(np.tile(synth.random_matrix(300, 257, 557)[:, :1], (1, 257)), 128)
