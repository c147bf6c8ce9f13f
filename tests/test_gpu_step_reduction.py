"""The per-step reductions at their edges against the plain form (one seed at a time, its own kernels): few and many
outputs, projection grids whose plan is copied to LDS or read in place, one and many ranges of S-norm partials, with and
without the support plan, on 4x4-block and general CSR storage. FP64; both orthogonalize fully, so levels and density
agree to 1e-9 of the largest."""
import numpy as np
import pytest

from paper_1307_3218_amd import lattice, mar

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", params=[0, 2], ids=["bsr", "csr"])
def system(request):
    s = lattice.generate(6, 5, 4, seed=6, check_spd=False)
    M = s.M - request.param
    ctx = mar.Context(s.H[:M, :M].tocsr(), s.S[:M, :M].tocsr())
    seeds = lattice.sample_seeds(M, 9, seed=1)
    ref = ctx.solve(seeds, 24, -0.4, 0.1, precision="fp64", form="plain", levels=True)
    yield ctx, seeds, ref
    ctx.close()


@pytest.mark.parametrize("block,wgs,support", [(1, 0, True), (2, 1, True), (16, 7, True), (16, 5000, True), (128, 0, True),
                                               (128, 5000, True), (128, 0, False), (128, 3, False), (8, 5000, False)])
def test_reductions(system, block, wgs, support):
    ctx, seeds, ref = system
    print(f"[step reduction block={block} wgs={wgs} support={support}]", flush=True)
    ctx.set_tuning(seed_block=block, proj_wgs=wgs, support=support)
    try:
        got = ctx.solve(seeds, 24, -0.4, 0.1, precision="fp64", levels=True)
    finally:
        ctx.set_tuning()
    assert np.array_equal(got.nu_eff, ref.nu_eff)
    for x, y in ((got.rho, ref.rho), (got.eps, ref.eps), (got.e_seed, ref.e_seed)):
        assert np.abs(x - y).max() <= 1e-9 * np.abs(y).max()
