"""The coupled-cluster kernel for spaces past LDS (12 and more active
orbitals), with several electrons of a spin: same-spin amplitudes and triples,
on both of its branches.  A call that holds few such tuples runs each on many
workgroups; one that holds many runs one workgroup per tuple.

Tolerance: both sides converge the amplitudes to 1e-11, energies to 1e-10; in
HF orbitals, converged to a gradient of 1e-10 on both sides, the (not
stationary) coupled-cluster energy follows to a few 1e-9 (bound 1e-8)."""
import itertools
import time

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


def test_some_large_tuples_in_a_list_run_batched(ws):
    """112 tuples of 11 orbitals, 56 of them past LDS (8+8 electrons): the
    call takes far less than the 56 sent one by one (a list of this length
    takes one launch for them; measured 0.04 of it)."""
    P = synth.small_problem(18, 9, 9, list(range(2, 10)), nvec=6, seed=4, vec_std=0.03, offdiag_std=0.02)
    tl = list(itertools.combinations(P.expansion_space(), 3))
    large = [t for t in tl if sum(p < 9 for p in t) == 1]
    tl = [t for t in tl if sum(p < 9 for p in t) == 0] + large
    assert len(tl) == 112 and len(large) == 56
    ctx = M.Context.from_problem(P, device=0, base_model=2)

    def seconds(lst):
        ctx.tuple_base(3, lst, ws)
        t0 = time.perf_counter()
        e = ctx.tuple_base(3, lst, ws)
        return time.perf_counter() - t0, e

    t_all, e_all = seconds(tl)
    t_one, e_one = seconds(large[:1])
    print(f"112 tuples {1e3 * t_all:.1f} ms, one large {1e3 * t_one:.1f} ms", flush=True)
    assert abs(e_all[56] - e_one[0]) <= TOL
    assert t_all < 0.5 * 56 * t_one
