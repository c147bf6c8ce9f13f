"""The delayed schedule's coefficient kernel at subspace dimensions where the partial sums of sixteen (nu > 2047) and of
eight wavefronts (nu > 2485) beside the vectors outgrow LDS: rows of three entries, in separate chains, so that every seed's subspace is exhausted
after its chain and the solve is quick."""
import numpy as np
import pytest
import scipy.sparse as sp

from oracle import mar_oracle as O
from paper_1307_3218_amd import mar

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nu", [2047, 2048, 2485, 2486])
def test_dimensions_past_two_thousand(nu):
    n, chain = 2500, 10
    rng = np.random.default_rng(1)
    off = rng.uniform(0.5, 1.0, n - 1)
    off[chain - 1::chain] = 0.0
    H = sp.diags([off, rng.uniform(-1.0, 1.0, n), off], [-1, 0, 1]).tocsr()
    H.eliminate_zeros()
    S = sp.eye(n).tocsr()
    seeds = np.array([3, 1207, 2499], dtype=np.int32)
    print(f"[coef nu={nu}]", flush=True)
    ctx = mar.Context(H, S)
    try:
        g = ctx.solve(seeds, nu, 0.0, 0.1, precision="fp64")
    finally:
        ctx.close()
    ref = O.solve(H, S, seeds, chain, 0.0, 0.1)
    assert g.nu_eff.max() <= chain and np.array_equal(g.nu_eff, ref.nu_eff)
    for j in seeds:
        sl = slice(H.indptr[j], H.indptr[j + 1])
        assert np.linalg.norm(g.rho[sl] - ref.rho[sl]) <= 1e-10 * np.linalg.norm(ref.rho[sl])
