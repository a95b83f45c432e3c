"""Coupled-cluster bases at the edges of the LDS kernel's sizes: one electron
of a spin, a spin without electrons, open shells with empty particle-hole sets,
the smallest spaces, two tuples per CU and one, and the border to the kernel
for larger spaces (11 and 12 active orbitals); several shapes in one call.
CCSD is exact for two electrons; the other energies are compared with the
oracle within its 1e-10 (both sides converge the amplitudes to 1e-11)."""
import itertools

import numpy as np
import pytest

import synth
from oracle import cc, fci

torch = pytest.importorskip("torch")
import paper_1905_02786_amd as M  # noqa: E402

pytestmark = pytest.mark.gpu
TOL = 1e-10


@pytest.fixture(scope="module")
def ws():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return M.workspace(2 << 30)


def problem(n, na, nb, ref):
    return synth.small_problem(n, na, nb, ref, nvec=6, seed=n + na, vec_std=0.05)


@pytest.mark.parametrize("na,nb,ref", [(1, 0, [0, 1]), (1, 1, [0, 1]), (2, 0, [0, 1, 2]), (2, 1, [0, 1, 2]),
                                       (3, 1, [1, 2, 3]), (3, 3, [2, 3])])
def test_shapes(ws, na, nb, ref):
    P = problem(6, na, nb, ref)
    X = P.expansion_space()
    ctx = M.Context.from_problem(P, device=0, base_model=2)
    for k in range(3):
        tl = list(itertools.combinations(X, k)) if k else [()]
        got = ctx.tuple_base(k, tl, ws)
        want = [fci.casci_energy(P, S) if na + nb <= 2 and len(P.ref) + k >= na else cc.base_energy(P, S) for S in tl]
        assert np.abs(got - np.array(want)).max() <= TOL


@pytest.mark.parametrize("nact", [8, 9, 10, 11, 12])
def test_two_electron_spaces(ws, nact):
    """CCSD = CASCI for two electrons, below, at and above the LDS border."""
    P = problem(nact + 1, 1, 1, [0, 1, 2])
    tl = [tuple(range(3, nact)), tuple(range(4, nact + 1))]
    ctx = M.Context.from_problem(P, device=0, base_model=2)
    got = ctx.tuple_base(nact - 3, tl, ws)
    assert np.abs(got - [fci.casci_energy(P, S) for S in tl]).max() <= TOL
