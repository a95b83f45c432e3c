"""sigma = H c at the edges of the electron counts (none, one, two electrons or
holes of a spin, a full shell) and of the vector counts, in workspaces that
hold all vectors, some and one, against the oracle's matvec.  The same
tolerance as the element-wise sigma parity tests: 1e-12 of the largest
element; the vectors' split over the workspace changes nothing, bitwise."""
import numpy as np
import pytest

import synth
from oracle import fci

torch = pytest.importorskip("torch")
import paper_1905_02786_amd as M  # noqa: E402

pytestmark = pytest.mark.gpu

CASES = [(n, na, nb) for n, na, nb in
         [(2, 1, 0), (2, 1, 1), (4, 2, 0), (4, 4, 2), (5, 3, 1), (6, 3, 3), (7, 5, 5), (8, 8, 7), (8, 7, 4), (9, 2, 1),
          (10, 3, 2), (12, 1, 1), (12, 11, 10), (12, 12, 12), (13, 2, 2), (13, 12, 11)]]


@pytest.fixture(scope="module")
def ws():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return M.workspace(1 << 30)


@pytest.mark.parametrize("n,na,nb", CASES)
@pytest.mark.parametrize("nvec", [1, 2, 5])
def test_sigma_at_edge_counts(ws, n, na, nb, nvec):
    P = synth.small_problem(n, na, nb, sorted({0, n - 1} | set(range(nb, na))), seed=n + na, e_const=0.7)
    S = tuple(P.expansion_space())
    sp = fci.cas_space(P, S)
    ctx = M.Context.from_problem(P, device=0)
    c = np.random.default_rng(7).standard_normal((nvec, sp.dim))
    ref = np.array([fci.matvec(P, sp, x) for x in c])
    ct = torch.tensor(c, device="cuda:0")
    sig = ctx.tuple_sigma(len(S), S, ct, ws).cpu().numpy()
    worst = np.abs(sig - ref).max() / max(1.0, np.abs(ref).max())
    print(f"n {n} electrons {na} {nb} dim {sp.dim} vectors {nvec}: {worst:.1e}", flush=True)
    assert worst <= 1e-12
    size = 1 << 16
    while True:   # the smallest power of two that is accepted: one vector, or a few
        try:
            one = ctx.tuple_sigma(len(S), S, ct, M.workspace(size)).cpu().numpy()
            break
        except M.MBEFCIError as ex:
            assert ex.code == -2 and size < 1 << 30
            size *= 2
    assert np.array_equal(one, sig)
    assert np.array_equal(ctx.tuple_sigma(len(S), S, ct, M.workspace(2 * size)).cpu().numpy(), sig)
