"""The coefficient kernel at the edges of its three forms (matrices in the registers of 4 or 8 wavefronts, or read in
chunks of 64 rows) against the plain form with its own schedule, and on a seed whose Krylov space is exhausted at once.
FP64; both orthogonalize fully, so density and energies (smooth functions of the subspaces) agree to 1e-9 of the largest."""
import numpy as np
import pytest
import scipy.sparse as sp

from paper_1307_3218_amd import lattice, mar

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def system():
    s = lattice.generate(4, 4, 3, mixed=True, seed=9, check_spd=False)
    # a block of four rows cut off from the rest: with diagonal blocks only: its seeds stop early
    keep = sp.diags((np.arange(s.M) >= 4).astype(float))
    cut = sp.diags((np.arange(s.M) < 4).astype(float))
    H, S = [(keep @ A @ keep + cut @ A @ cut).tocsr() for A in (s.H, s.S)]
    ctx = mar.Context(H, S)
    yield ctx
    ctx.close()


@pytest.mark.parametrize("nu", [1, 2, 31, 32, 33, 63, 64, 65, 128, 130])
def test_forms(system, nu):
    ctx, seeds = system, np.array([1, 4, 700, 701, 1500], dtype=np.int32)
    print(f"[coef nu={nu}]", flush=True)
    ref = ctx.solve(seeds, nu, -0.4, 0.1, precision="fp64", form="plain")
    ctx.set_tuning(seed_block=8)
    try:
        got = ctx.solve(seeds, nu, -0.4, 0.1, precision="fp64")
    finally:
        ctx.set_tuning()
    assert np.array_equal(got.nu_eff, ref.nu_eff) and (nu < 5 or got.nu_eff[0] <= 4)
    for x, y in ((got.rho, ref.rho), (got.n_seed, ref.n_seed), (got.e_seed, ref.e_seed)):
        assert np.abs(x - y).max() <= 1e-9 * np.abs(y).max()
