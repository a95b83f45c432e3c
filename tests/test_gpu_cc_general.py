"""The coupled-cluster kernel for spaces past LDS (12 and more active
orbitals), with several electrons of a spin: same-spin amplitudes and triples,
on both of its branches.  A call that holds few such tuples runs each on many
workgroups; one that holds many runs one workgroup per tuple.

Tolerance: both sides converge the amplitudes to 1e-11, energies to 1e-10; in
HF orbitals, converged to a gradient of 1e-10 on both sides, the (not
stationary) coupled-cluster energy follows to a few 1e-9 (bound 1e-8)."""
import itertools

import numpy as np
import pytest

import synth
from oracle import cc, hf

torch = pytest.importorskip("torch")
import paper_1905_02786_amd as M  # noqa: E402

pytestmark = pytest.mark.gpu
TOL = 1e-10


@pytest.fixture(scope="module")
def ws():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return M.workspace(4 << 30)


def test_one_tuple_on_many_workgroups(ws):
    P = synth.small_problem(12, 2, 2, [1, 2], nvec=5, seed=7, offdiag_std=0.05)
    X = tuple(P.expansion_space())
    got = M.Context.from_problem(P, device=0, base_model=2).tuple_base(len(X), [X], ws)[0]
    assert abs(got - cc.base_energy(P, X)) <= TOL
    _, Q, _ = hf.hf_problem(P)
    ctx = M.Context.from_problem(P, device=0, base_model=3)
    ctx.hf(ws)
    assert abs(ctx.tuple_base(len(X), [X], ws)[0] - cc.base_energy(Q, X, triples=True)) <= 1e-8


@pytest.mark.parametrize("na,nb,model", [(3, 3, 3), (4, 3, 2)])
def test_many_tuples_one_workgroup_each(ws, na, nb, model):
    """84 tuples of 12 orbitals in one call against the same ones sent three
    at a time (many workgroups each); closed shell with triples, open shell."""
    P = synth.small_problem(18, na, nb, list(range(1, 10)), nvec=6, seed=4, vec_std=0.05)
    ctx = M.Context.from_problem(P, device=0, base_model=model)
    if model == 3:
        ctx.hf(ws)
    tl = list(itertools.combinations(P.expansion_space(), 3))
    assert len(tl) == 84   # (a quarter of a cooperative launch is at most 64 workgroups)
    got = ctx.tuple_base(3, tl, ws)
    few = np.concatenate([ctx.tuple_base(3, tl[i:i + 3], ws) for i in range(0, 84, 3)])
    assert np.abs(got - few).max() <= TOL
