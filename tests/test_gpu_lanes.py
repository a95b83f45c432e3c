"""Shape classes solved at the same time (a workspace that holds several) and
one after the other (a workspace of one class's size, or of one tuple's): the
same energies, statuses and iterations, bitwise, for lists with one to five
classes, tuples that need the second pass, several threads with their own streams
and contexts, and gradients up to the order of the device's atomic adds.  A
workspace too small for one tuple is refused as before."""
import itertools
import threading

import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
import paper_1905_02786_amd as M  # noqa: E402

pytestmark = pytest.mark.gpu

PROBLEMS = {
    "plain": lambda: synth.config_plain(0),
    "openshell": lambda: synth.small_problem(10, 5, 4, [4, 5], nvec=8, seed=3, e_const=0.5),
}


@pytest.fixture(scope="module")
def ws():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return M.workspace(2 << 30)


def solve(ctx, k, tl, w, **kw):
    e, st = ctx.solve_tuples(k, tl, w, **kw)
    s = ctx.stats()
    return e, st, (s["iterations_total"], s["second_pass"])


@pytest.mark.parametrize("whole", [0, 1225])
@pytest.mark.parametrize("name", sorted(PROBLEMS))
@pytest.mark.parametrize("k", [0, 1, 2, 3, 4])
def test_classes_together_and_apart(ws, name, k, whole):
    P = PROBLEMS[name]()
    tl = list(itertools.combinations(P.expansion_space(), k))
    ctx = M.Context.from_problem(P, device=0, whole_dim=whole)
    mn, want = ctx.workspace_query(k, tl)
    ref = solve(ctx, k, tl, ws)
    for nbytes in (want, mn):
        got = solve(ctx, k, tl, M.workspace(nbytes))
        print(f"{name} order {k} whole {whole}: {len(tl)} tuples in {nbytes} bytes", flush=True)
        assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1], ref[1]) and got[2] == ref[2]
    with pytest.raises(M.MBEFCIError) as ex:
        ctx.solve_tuples(k, tl, M.workspace(mn // 2))
    assert ex.value.code == -2


@pytest.mark.parametrize("whole", [0, 1225])
def test_second_pass(ws, whole):
    # every tuple fails after one iteration and is solved again
    P = PROBLEMS["plain"]()
    tl = list(itertools.combinations(P.expansion_space(), 3))
    ctx = M.Context.from_problem(P, device=0, whole_dim=whole, max_iter=1, pspace=1)
    mn, _ = ctx.workspace_query(3, tl)
    ref = solve(ctx, 3, tl, M.workspace(mn))
    got = solve(ctx, 3, tl, ws)
    assert ref[2][1] > 0
    assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1], ref[1]) and got[2] == ref[2]


def test_threads_and_streams(ws):
    P = PROBLEMS["openshell"]()
    tl = list(itertools.combinations(P.expansion_space(), 3))
    ref = M.Context.from_problem(P, device=0).solve_tuples(3, tl, ws)[0]
    got = [None] * 4

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            ctx = M.Context.from_problem(P, device=0)
            w = M.workspace(256 << 20)
            for _ in range(3):
                got[i] = ctx.solve_tuples(3, tl, w)[0]

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(got))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for e in got:
        assert np.array_equal(e, ref)


def test_gradient(ws):
    P = PROBLEMS["plain"]()
    g = []
    for w in (ws, M.workspace(24 << 20)):
        ctx = M.Context.from_problem(P, device=0, gradient=1, max_order=4)
        res, h = ctx.run(w, keep=True)
        g.append((res.total,) + tuple(ctx.backward(h, w)))
    assert g[0][0] == g[1][0]
    for a, b in zip(g[0][1:], g[1][1:]):
        assert np.abs(a - b).max() <= 1e-12


def test_repeats_are_bitwise(ws):
    # every sigma form of the plain expansion beside the others: a wave that
    # falls behind must not change what it or its neighbours read
    P = PROBLEMS["plain"]()
    lists = [(k, list(itertools.combinations(P.expansion_space(), k))) for k in (5, 6, 7)]
    ctx = M.Context.from_problem(P, device=0)
    small = M.workspace(8 << 20)   # (one tuple of the largest, in the form that needs most)
    ref = [ctx.solve_tuples(k, tl, small)[0] for k, tl in lists]
    for rep in range(60):
        for (k, tl), r in zip(lists, ref):
            assert np.array_equal(ctx.solve_tuples(k, tl, ws)[0], r), (rep, k)
