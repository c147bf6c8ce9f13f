"""Products in general CSR storage: rows of 1 to 40 entries (one and several groups of eight), an S on H's pattern (one
pass for both) and on a part of it, and block widths from one seed to a wavefront per row, against the plain form with
one seed at a time. FP64; both orthogonalize fully, so density and energies agree to 1e-9 of the largest."""
import numpy as np
import pytest
import scipy.sparse as sp

from paper_1307_3218_amd import mar

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", params=[True, False], ids=["same", "part"])
def system(request):
    n = 997
    rng = np.random.default_rng(5)
    r, c = rng.integers(0, n, 2600), rng.integers(0, n, 2600)
    r, c = np.concatenate([r, np.full(39, 7)]), np.concatenate([c, rng.choice(np.arange(8, n), 39, replace=False)])
    keep = (r != c) & (r != 3) & (c != 3)          # row 3 has its diagonal entry alone
    A = sp.coo_matrix((rng.standard_normal(keep.sum()), (r[keep], c[keep])), shape=(n, n)).tocsr()
    A.sum_duplicates()
    H = (A + A.T + sp.diags(rng.standard_normal(n))).tocsr()
    H.sort_indices()
    S = H.copy()
    i = np.repeat(np.arange(n), np.diff(H.indptr))
    S.data = np.where(i == H.indices, 1.0, 0.01)
    if not request.param:
        S.data[(i != H.indices) & ((i + H.indices) % 3 == 0)] = 0.0
        S.eliminate_zeros()
    ctx = mar.Context(H, S)
    seeds = np.r_[0:9, 300:420].astype(np.int32)
    print(f"[csr products] rows of {np.diff(H.indptr).min()} to {np.diff(H.indptr).max()}, S {S.nnz} of {H.nnz}", flush=True)
    yield ctx, seeds, ctx.solve(seeds, 14, 0.2, 0.3, precision="fp64", form="plain")
    ctx.close()


@pytest.mark.parametrize("prec,block", [("fp64", 1), ("fp64", 2), ("fp64", 8), ("fp64", 64), ("fp64", 128), ("fp32", 2),
                                        ("fp32", 4), ("fp32", 256)])
def test_products(system, prec, block):
    ctx, seeds, ref = system
    ctx.set_tuning(seed_block=block)
    try:
        got = ctx.solve(seeds, 14, 0.2, 0.3, precision=prec)
    finally:
        ctx.set_tuning()
    assert np.array_equal(got.nu_eff, ref.nu_eff)
    tol = 1e-9 if prec == "fp64" else 2e-5
    for x, y in ((got.rho, ref.rho), (got.n_seed, ref.n_seed), (got.e_seed, ref.e_seed)):
        assert np.abs(x - y).max() <= tol * np.abs(y).max()
