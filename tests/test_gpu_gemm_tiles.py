"""H_eff beyond the one-launch sizes at the edges of its GEMM tiles: row, column and depth remainders of the
32 x 32 tile, odd and even sizes (element and pair loads), a bond past the line where larger tiles take over,
and the batched engine with every grouped GEMM on the 32 x 32 tile."""
import numpy as np
import pytest

import oracle
from gpu_common import ctx, env_pair, to_dev
from test_gpu_batch import _chains, _check, _run

pytestmark = pytest.mark.gpu

SHAPES = [(1, 81), (2, 200), (31, 97), (33, 95), (64, 96), (65, 127), (193, 1), (194, 2), (193, 129), (224, 160),
          (520, 505)]
MODELS = [(0, [1.0, 1.0, 0.0]), (1, [1.0, 0.241]), (2, [1.0, 0.7])]


@pytest.mark.parametrize("chl,chr_", SHAPES)
@pytest.mark.parametrize("model,params", MODELS)
def test_small_tiles_match_oracle(chl, chr_, model, params):
    """Tolerances as for the general sizes: 1e-14 (FP64) and 2e-6 (FP32) of the largest possible entry."""
    import paper_2604_03960_amd as tna
    W, L, R, th = env_pair(model, params, chl, chr_, 900 + 3 * chl + chr_)
    args = [to_dev(x) for x in (L, W[1], W[2], R, th)]
    ref = oracle.heff_apply(L, W[1], W[2], R, th)
    scale = np.abs(L).max() * np.abs(R).max() * np.abs(th).max() * max(chl, chr_) * 8
    for prec, tol in ((tna.HEFF_F64, 1e-14), (tna.HEFF_F32, 2e-6)):
        got = ctx().heff_apply(*args, prec=prec).cpu().numpy()
        assert np.abs(got - ref).max() <= tol * scale


@pytest.mark.parametrize("prec", [0, 1])
def test_batch_on_the_small_tile_matches_oracle(prec, tmp_path):
    """The autotuner table forced to the 32 x 32 tile, chi pinned at 40: short and grouped paths."""
    import paper_2604_03960_amd as tna
    table = tmp_path / "tiles.txt"
    table.write_text("".join(f"{op} {b} 32\n" for op in range(7) for b in range(64)))
    tna.autotune_clear()
    tna.autotune_load(str(table))
    try:
        chains = _chains(3, (14, 16), seed=7)
        Es, logs, stats = _run(chains, 2, prec, chi_max=40, chi_min=40)
        assert stats["graph_launches"] > 0 and stats["autotune_entries"] == 7 * 64
        _check(chains, 2, prec, 40, Es, logs, chi_min=40)
    finally:
        tna.autotune_clear()
