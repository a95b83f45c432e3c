"""The Davidson iteration's per-tuple kernels at the edges of their sizes: the
projected eigenproblem (16 lanes a row group up to 12 vectors, 32 above, one
to three basis vectors, restarts that keep one or two vectors) and the P space
(1 to 128 determinants, the whole CAS, sizes around the kernels' 32 and 64
steps), batched and in whole-tuple mode, against the oracle's CASCI energies.
The tolerance is the parity tests' 1e-10: the residual bound of 1e-6 squared
over the smallest gap of these spaces (0.01) is 1e-10, and is not reached from
one iteration to the next."""
import itertools

import numpy as np
import pytest

import synth
from oracle import fci

torch = pytest.importorskip("torch")
import paper_1905_02786_amd as M  # noqa: E402

pytestmark = pytest.mark.gpu
TOL = 1e-10


@pytest.fixture(scope="module")
def ws():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return M.workspace(1 << 30)


@pytest.fixture(scope="module")
def case():
    P = synth.small_problem(8, 4, 3, [3, 4], nvec=8, seed=11)
    X = P.expansion_space()
    tuples = {k: list(itertools.combinations(X, k))[:6] for k in (0, 1, 2, 3, 4)}
    return P, tuples, {k: np.array([fci.casci_energy(P, S) for S in t]) for k, t in tuples.items()}


@pytest.mark.parametrize("whole", [0, 1225])
@pytest.mark.parametrize("space,keep,psp", [(2, 1, 0), (3, 2, 8), (4, 2, 128), (11, 1, 31), (12, 2, 1), (12, 2, 32),
                                            (12, 2, 33), (13, 2, 64), (16, 1, 65), (17, 2, 127), (32, 2, 128)])
def test_subspace_and_p_space_sizes(ws, case, whole, space, keep, psp):
    P, tuples, ref = case
    ctx = M.Context.from_problem(P, device=0, whole_dim=whole, max_space=space, restart_keep=keep, pspace=psp,
                                 max_iter=3000)
    worst = 0.0
    for k, t in tuples.items():
        e, st = ctx.solve_tuples(k, t, ws)
        assert (st == 0).all()
        worst = max(worst, float(np.abs(e - ref[k]).max()))
    print(f"space {space} keep {keep} psp {psp} whole {whole}: max |d eps| {worst:.1e}", flush=True)
    assert worst <= TOL
