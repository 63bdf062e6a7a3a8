"""The single-workgroup Lanczos with its basis in registers, at the edges of its forms: theta of 256, 512 and
1024 elements and just past them, fewer and more vectors than the registers hold, both precisions."""
import numpy as np
import pytest

import oracle
import synth
from gpu_common import ctx
from test_gpu_batch import _chains, _check, _run
from test_gpu_dmrg import _compare_amb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("chi", [8, 9, 11, 12, 16, 17])
@pytest.mark.parametrize("prec", [0, 1])
def test_basis_forms_match_oracle(chi, prec):
    """chi pinned: middle bonds have 4 chi^2 elements, the edge bonds run the shorter forms.  Tolerances of the
    batched sweeps."""
    chains = _chains(3, (10, 12), seed=20 + chi)
    Es, logs, stats = _run(chains, 2, prec, chi_max=chi, chi_min=chi)
    assert stats["small_launches"] > 0
    _check(chains, 2, prec, chi, Es, logs, chi_min=chi)


@pytest.mark.parametrize("chi,its", [(8, 100), (11, 90), (16, 41), (16, 70)])
def test_more_vectors_than_registers(chi, its):
    """A fixed number of iterations, past the 40 (16 x 16) and 80 (11 x 11) vectors kept, at the tolerance of
    the fixed-iteration sweeps."""
    import paper_2604_03960_amd as tna
    N = 12
    W = oracle.mpo(oracle.MODEL_XXZ, N, [1.0, 0.8, 0.0])
    A, c0, _ = synth.random_mps(N, 2, chi, seed=31)
    pp = (2.0, 0.1, 0.5, 1.0, 0.3, chi, chi)
    ro = oracle.dmrg_run(W, A, c0, oracle.pid_params(*pp), 1, fixed_iters=its, fixed_chi=chi)
    dm = tna.Dmrg(ctx(), W, A, c0, tna.pid_params(*pp), fixed_iters=its, fixed_chi=chi)
    E, recs, _ = dm.sweep()
    assert dm.stats()["small_launches"] > 0
    assert max(g["lanczos_iters"] for g in recs) == its
    amb = _compare_amb(ro, np.array([E]), recs, 1e-10, N)
    assert abs(E - ro["E"][0]) / N <= 1e-10 + amb


@pytest.mark.parametrize("model,params", [(0, [1.0, 0.8, 0.0]), (1, [1.0, 0.241]), (2, [1.0, 1.3])])
@pytest.mark.parametrize("chi", [11, 12, 14])
def test_mixing_forms(model, params, chi):
    """Both forms of the mixing (121 columns a chunk and more) at every MPO bond dimension in use, twelve
    matvecs a visit, at the tolerance of the fixed-iteration sweeps."""
    import paper_2604_03960_amd as tna
    N = 10
    W = oracle.mpo(model, N, params)
    A, c0, _ = synth.random_mps(N, 2, chi, seed=77)
    pp = (2.0, 0.1, 0.5, 1.0, 0.3, chi, chi)
    ro = oracle.dmrg_run(W, A, c0, oracle.pid_params(*pp), 1, fixed_iters=12, fixed_chi=chi)
    dm = tna.Dmrg(ctx(), W, A, c0, tna.pid_params(*pp), fixed_iters=12, fixed_chi=chi)
    E, recs, _ = dm.sweep()
    assert dm.stats()["small_launches"] > 0
    amb = _compare_amb(ro, np.array([E]), recs, 1e-10, N)
    assert abs(E - ro["E"][0]) / N <= 1e-10 + amb
