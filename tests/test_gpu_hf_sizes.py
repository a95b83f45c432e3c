"""Fock and Hessian kernels of mbefci_hf at the edges of their sizes: one
occupied orbital, one virtual, odd orbital counts below and above the block
widths, against the oracle's Hartree-Fock.  Tolerances as in test_gpu_hf: both
sides converge the orbital gradient to 1e-10, the energy is stationary (1e-10)
and the orbitals follow to 1e-10 over the smallest Hessian estimate (1e-6)."""
import numpy as np
import pytest

import synth
from oracle import hf

torch = pytest.importorskip("torch")
import paper_1905_02786_amd as M  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,no", [(2, 1), (3, 1), (9, 8), (16, 5), (17, 4), (33, 6)])
def test_hf_sizes(n, no):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    diag = np.concatenate([np.linspace(-1.3, -0.5, no), np.linspace(0.2, 2.5, n - no)])
    h, eri = synth.random_hamiltonian(diag, 0.05, 2 * n, np.sqrt(0.05 / (2 * n)), 7)
    P = synth.Problem("hf-sizes", h, eri, no, no, 0, [no - 1])
    e_ref, C_ref, eps = hf.rhf(P)
    ctx = M.Context.from_problem(P, device=0)
    out = ctx.hf(M.workspace(1 << 26))
    assert abs(out["energy"] - e_ref) <= 1e-10
    U = out["U"]
    assert np.abs(U.T @ U - np.eye(n)).max() <= 1e-12
    sg = np.sign(np.sum(U * C_ref, axis=0))
    print(f"n {n} occupied {no}: |U - U_ref| {np.abs(U * sg - C_ref).max():.1e}", flush=True)
    assert np.abs(U * sg - C_ref).max() <= 1e-6
