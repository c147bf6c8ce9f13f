"""The subspace eigensolve by Householder reduction and implicit QL (k_tri, k_tri_big, k_ql) against the oracle's
LAPACK result, over the edges of its register tiles (16 columns, 32 rows), the step to the version with A in global
memory (nu > 128), subspaces cut short by a breakdown, and rows of up to 60 entries (further rows of the reduction).

Bars: those of the FP64 form, 1e-10 relative per rho column and for E_band, levels to 1e-10 of the spectral scale,
weights summing to one; the Jacobi iteration (asked for with a sweep cap) agrees to the same bars.
"""
import numpy as np
import pytest
import scipy.sparse as sp

from oracle import mar_oracle as O
from paper_1307_3218_amd import lattice, mar

pytestmark = pytest.mark.gpu

KT, MU = 0.1, -0.3


def _check(H, S, seeds, nu):
    ctx = mar.Context(H, S)
    try:
        print(f"[eig ql] M={H.shape[0]} row {int(np.diff(H.indptr).max())} nu={nu}", flush=True)
        g = ctx.solve(seeds, nu, MU, KT, levels=True)
        ctx.set_tuning(eig_max_sweeps=40)
        jac = ctx.solve(seeds, nu, MU, KT, levels=True)
    finally:
        ctx.close()
    ref = O.solve(H, S, seeds, nu, MU, KT)
    assert np.array_equal(g.nu_eff, ref.nu_eff)
    assert abs(g.e_band - ref.e_band) <= 1e-10 * abs(ref.e_band)
    scale = max(np.abs(e).max() for e in ref.eps)
    for s, j in enumerate(seeds):
        m, sl = g.nu_eff[s], slice(H.indptr[j], H.indptr[j + 1])
        norm = np.linalg.norm(ref.rho[sl])
        assert np.linalg.norm(g.rho[sl] - ref.rho[sl]) <= 1e-10 * norm
        assert np.linalg.norm(g.rho[sl] - jac.rho[sl]) <= 1e-10 * norm
        assert np.abs(np.sort(g.eps[s, :m]) - ref.eps[s]).max() <= 1e-10 * scale
        assert np.all(g.eps[s, m:] == 0.0) and np.all(g.weight[s, m:] == 0.0)
        assert abs(g.weight[s].sum() - 1.0) <= 1e-10


@pytest.fixture(scope="module")
def cell():
    s = lattice.generate(4, 3, 3, mixed=True, seed=2)
    return s.H.tocsr(), s.S.tocsr()


@pytest.mark.parametrize("nu", [1, 2, 3, 4, 15, 16, 17, 32, 33, 64, 65, 96, 97, 112, 128, 129, 140, 300])
def test_dimensions(cell, nu):
    H, S = cell
    _check(H, S, np.arange(3, H.shape[0], 211, dtype=np.int32), nu)


def test_subspaces_cut_short():
    """nu = M and beyond a seed's reach: every breakdown length from 4 rows (a block alone) to the whole cell."""
    s = lattice.generate(2, 1, 1)
    H, S = s.H.tocsr(), s.S.tocsr()
    _check(H, S, np.arange(0, s.M, 5, dtype=np.int32), s.M)
    A = sp.block_diag([H, 2.0 * sp.eye(4) + sp.csr_matrix(np.ones((4, 4)))]).tocsr()
    B = sp.block_diag([S, sp.eye(4)]).tocsr()
    A.sort_indices()
    B.sort_indices()
    _check(A, B, np.array([0, s.M, s.M + 3], dtype=np.int32), 40)


@pytest.mark.parametrize("nu", [20, 40, 70, 97, 128, 150])
def test_long_rows(nu):
    rng = np.random.default_rng(5)
    nb = 100
    P = np.eye(nb, dtype=bool)
    for i in range(nb):
        for j in rng.choice(nb, size=9, replace=False):
            if P[i].sum() < 15 and P[j].sum() < 15:
                P[i, j] = P[j, i] = True
    rows, cols = np.nonzero(np.kron(P, np.ones((4, 4))))
    A, B = rng.standard_normal((4 * nb, 4 * nb)), 0.005 * rng.standard_normal((4 * nb, 4 * nb))
    H = sp.csr_matrix(((A + A.T)[rows, cols], (rows, cols)), shape=A.shape)
    S = sp.csr_matrix(((B + B.T + np.eye(4 * nb))[rows, cols], (rows, cols)), shape=A.shape)
    assert np.diff(H.indptr).max() == 60
    _check(H, S, np.arange(0, 4 * nb, 57, dtype=np.int32), nu)
