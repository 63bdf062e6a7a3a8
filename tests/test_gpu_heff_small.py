"""The one-launch H_eff of short bonds at its edges: row and column remainders of its tiles, the limits where
the general path takes over, every MPO bond dimension in use, both precisions, and results written over an
input that has been read."""
import numpy as np
import pytest

import oracle
from gpu_common import ctx, env_pair, to_dev

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1), (2, 80), (3, 17), (4, 4), (5, 79), (15, 16), (17, 15), (192, 3), (192, 80), (193, 80), (40, 81)]
MODELS = [(0, [1.0, 1.0, 0.0]), (1, [1.0, 0.241]), (2, [1.0, 0.7])]


@pytest.mark.parametrize("chl,chr_", SHAPES)
@pytest.mark.parametrize("model,params", MODELS)
def test_short_bonds_match_oracle(chl, chr_, model, params):
    """Tolerances as for the general sizes: 1e-14 (FP64) and 2e-6 (FP32) of the largest possible entry."""
    import paper_2604_03960_amd as tna
    W, L, R, th = env_pair(model, params, chl, chr_, 500 + 3 * chl + chr_)
    args = [to_dev(x) for x in (L, W[1], W[2], R, th)]
    ref = oracle.heff_apply(L, W[1], W[2], R, th)
    scale = np.abs(L).max() * np.abs(R).max() * np.abs(th).max() * max(chl, chr_) * 8
    for prec, tol in ((tna.HEFF_F64, 1e-14), (tna.HEFF_F32, 2e-6)):
        got = ctx().heff_apply(*args, prec=prec).cpu().numpy()
        assert np.abs(got - ref).max() <= tol * scale


@pytest.mark.parametrize("prec", [0, 1])
def test_result_over_an_input_already_read(prec):
    """The result may be written over the left environment's memory: the same bits as into its own."""
    W, L, R, th = env_pair(0, [1.0, 1.0, 0.0], 24, 20, 9)
    dL, W1, W2, dR, dth = [to_dev(x) for x in (L, W[1], W[2], R, th)]
    want = ctx().heff_apply(dL, W1, W2, dR, dth, prec=prec).clone()
    over = dL.view(-1)[:dth.numel()].view(dth.shape)
    got = ctx().heff_apply(dL, W1, W2, dR, dth, prec=prec, out=over)
    assert (got == want).all()


@pytest.mark.parametrize("chl,chr_", [(192, 32), (193, 32), (192, 33), (64, 48), (65, 48), (64, 49)])
def test_both_sides_of_the_line(chl, chr_):
    """The longest bonds of the one-launch form and the first of the general one: a result written over an
    input takes the general path, and both give the same bits."""
    W, L, R, th = env_pair(1, [1.0, 0.241], chl, chr_, 60)
    dL, W1, W2, dR, dth = [to_dev(x) for x in (L, W[1], W[2], R, th)]
    got = ctx().heff_apply(dL, W1, W2, dR, dth).clone()
    ref = oracle.heff_apply(L, W[1], W[2], R, th)
    scale = np.abs(L).max() * np.abs(R).max() * np.abs(th).max() * max(chl, chr_) * 8
    assert np.abs(got.cpu().numpy() - ref).max() <= 1e-14 * scale
    over = dL.view(-1)[:dth.numel()].view(dth.shape)
    assert (got == ctx().heff_apply(dL, W1, W2, dR, dth, out=over)).all()
