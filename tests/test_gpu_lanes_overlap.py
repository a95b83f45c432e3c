"""Shape classes that fit the workspace side by side are under way at the same
time: the classes' batches, each timed from its start to its end, then add up
to more than the call took.  In a workspace of one tuple they follow each other
and cannot."""
import itertools

import pytest

import synth

torch = pytest.importorskip("torch")
import paper_1905_02786_amd as M  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [3, 5])
def test_classes_overlap(k):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    P = synth.config_plain(0)
    tl = list(itertools.combinations(P.expansion_space(), k))
    ctx = M.Context.from_problem(P, device=0, whole_dim=0)
    mn, want = ctx.workspace_query(k, tl)
    wall = {}
    for name, nbytes in (("several", 2 << 30), ("one", mn)):
        w = M.workspace(nbytes)
        ctx.solve_tuples(k, tl, w)   # (tables, the choice of sigma form)
        ctx.solve_tuples(k, tl, w)
        cs = ctx.class_stats()
        assert len(cs) >= 3 and sum(c["tuples"] for c in cs) == len(tl)
        wall[name] = sum(c["wall_ms"] for c in cs), ctx.stats()["solve_ms"]
        print(f"order {k}, {name}: {len(cs)} classes, batches {wall[name][0]:.2f} ms, call {wall[name][1]:.2f} ms",
              flush=True)
    assert wall["several"][0] > wall["several"][1]
    assert wall["one"][0] <= wall["one"][1]
