"""H_eff whose last product has just under or just over the number of 64 x 64 tiles (440) from which that tile is
taken instead of the 32 x 32 one."""
import numpy as np
import pytest

import oracle
from gpu_common import ctx, env_pair, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("chl,chr_", [(432, 1000), (431, 1023), (433, 1024), (447, 1023), (466, 1050)])
@pytest.mark.parametrize("prec,tol", [(0, 1e-12), (1, 1e-5)])
def test_both_sides_of_the_tile_line(chl, chr_, prec, tol):
    """432 (even and odd sizes), 448 (likewise) and 510 tiles: 24 elements against the oracle's definition, tolerance
    relative to the RMS of the result as at chi = 1024."""
    W, L, R, th = env_pair(2, [1.0, 0.7], chl, chr_, 70)
    L, R = L / chl, R / chr_
    out = ctx().heff_apply(*[to_dev(x) for x in (L, W[1], W[2], R, th)], prec=prec).cpu().numpy()
    rms = np.sqrt(np.mean(out ** 2))
    rng = np.random.default_rng(chl)
    for _ in range(24):
        idx = tuple(int(rng.integers(k)) for k in out.shape)
        assert abs(out[idx] - oracle.heff_element(L, W[1], W[2], R, th, idx)) <= tol * rms
