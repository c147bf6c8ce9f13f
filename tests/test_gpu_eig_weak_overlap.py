"""The subspace eigensolve on a basis with a weak overlap: A = K^T H K then has entries of the overlap's size below the
subdiagonal of every column, far smaller than the subdiagonal and far larger than rounding, and the reduction to
tridiagonal form (k_tri to nu = 128, k_tri_big above) must not take them for zeros.

Bars: those of the FP64 form against the oracle, 1e-10 of the spectral scale per level, 1e-10 relative per rho column.
"""
import numpy as np
import pytest
import scipy.sparse as sp

from oracle import mar_oracle as O
from paper_1307_3218_amd import lattice, mar

pytestmark = pytest.mark.gpu

KT, MU = 0.1, -0.3


@pytest.mark.parametrize("overlap", [1e-7, 1e-8, 3e-9, 1e-9, 1e-11])
@pytest.mark.parametrize("nu", [30, 64, 100, 129])
def test_small_entries_below_the_subdiagonal(nu, overlap):
    s = lattice.generate(4, 3, 3, mixed=True, seed=2)
    H, S = s.H.tocsr(), s.S.tocsr()
    off = S - sp.diags(S.diagonal())
    S = (sp.eye(s.M) + off * (overlap / np.abs(off.data).max())).tocsr()
    S.sort_indices()
    seeds = np.arange(3, s.M, 211, dtype=np.int32)
    ref = O.solve(H, S, seeds, nu, MU, KT)
    scale = max(np.abs(e).max() for e in ref.eps)
    ctx = mar.Context(H, S)
    try:
        g = ctx.solve(seeds, nu, MU, KT, levels=True)
    finally:
        ctx.close()
    assert np.array_equal(g.nu_eff, ref.nu_eff)
    lev = max(np.abs(np.sort(g.eps[i, :m]) - ref.eps[i]).max() for i, m in enumerate(g.nu_eff)) / scale
    col = max(np.linalg.norm(g.rho[sl] - ref.rho[sl]) / np.linalg.norm(ref.rho[sl])
              for sl in (slice(H.indptr[j], H.indptr[j + 1]) for j in seeds))
    print(f"[weak overlap] nu={nu} overlap {overlap:.0e}: levels {lev:.1e}, rho columns {col:.1e}", flush=True)
    assert lev <= 1e-10 and col <= 1e-10
