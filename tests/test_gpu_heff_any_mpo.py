"""H_eff with MPO bond dimensions and site dimensions beyond those of the built-in models (any D d^2 <= 32): the
one-launch form (192 x 32 and 64 x 48 are its longest bonds) and the mixing kernel with run-time channel counts."""
import numpy as np
import pytest

import oracle
import synth
from gpu_common import ctx, to_dev

pytestmark = pytest.mark.gpu

MPOS = [(2, 1), (2, 2), (2, 4), (2, 6), (2, 7), (3, 1), (3, 2), (3, 3), (4, 1), (4, 2), (1, 5), (1, 32)]  # d, D
SHAPES = [(1, 1), (5, 7), (17, 33), (64, 48), (64, 49), (192, 32), (193, 32)]


def _operands(d, D, chl, chr_):
    seed = 1000 * d + 40 * D + chl + chr_
    shapes = [(chl, D, chl), (D, D, d, d), (D, D, d, d), (chr_, D, chr_), (chl, d, d, chr_)]
    return [synth.normal(seed + i, int(np.prod(s))).reshape(s) for i, s in enumerate(shapes)]


def _bound(d, D, chl, chr_, args, prec):
    """n roundings of the sum of absolute products: the lengths of the three sums and of M's, plus one per factor; in
    FP32 the factors are rounded first.  Twice: the oracle has its own."""
    n = chl + D + D * d * d + D * chr_ + 6
    return 2 * n * 2.0 ** (-53 if prec == 0 else -24) * oracle.heff_apply(*[np.abs(x) for x in args])


@pytest.mark.parametrize("chl,chr_", SHAPES)
@pytest.mark.parametrize("d,D", MPOS)
def test_any_mpo_matches_oracle(d, D, chl, chr_):
    args = _operands(d, D, chl, chr_)
    ref = oracle.heff_apply(*args)
    dev = [to_dev(x) for x in args]
    for prec in (0, 1):
        got = ctx().heff_apply(*dev, prec=prec).cpu().numpy()
        assert np.all(np.abs(got - ref) <= _bound(d, D, chl, chr_, args, prec))


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("chl,chr_", [(5, 7), (64, 48), (192, 32)])
@pytest.mark.parametrize("D", [1, 2, 3, 4, 5, 6, 7, 8])
def test_one_launch_and_general_path_give_the_same_bits(D, chl, chr_, prec):
    """A result written over an input takes the general path."""
    import torch
    L, W1, W2, R, th = [to_dev(x) for x in _operands(2, D, chl, chr_)]
    got = ctx().heff_apply(L, W1, W2, R, th, prec=prec)
    buf = torch.zeros(max(L.numel(), th.numel()), dtype=torch.float64, device="cuda")
    over = buf[:L.numel()].view(L.shape)
    over.copy_(L)
    assert (got == ctx().heff_apply(over, W1, W2, R, th, prec=prec, out=buf[:th.numel()].view(th.shape))).all()
