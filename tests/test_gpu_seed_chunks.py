"""One workgroup per seed where a projection takes the rows in one, two (unequal) and several chunks, with part of the
basis, down to a single vector of a group of four, in memory, against the seed blocks' kernels. Both orthogonalize fully:
density and energies agree to 1e-9 (FP64) and 2e-5 (FP32) of the largest."""
import numpy as np
import pytest

from paper_1307_3218_amd import lattice, mar

pytestmark = pytest.mark.gpu


# rows 512 (one chunk in FP64), 576 and 1056 (two and three), 2048 (four; 6 of 7 and of 30 vectors in LDS), 3072 (six)
@pytest.mark.parametrize("cells,nu,prec", [((4, 4, 1), 40, "fp64"), ((6, 3, 1), 33, "fp64"), ((11, 3, 1), 21, "fp64"),
                                           ((4, 4, 4), 7, "fp64"), ((4, 4, 4), 30, "fp64"), ((6, 4, 4), 12, "fp64"),
                                           ((6, 4, 4), 50, "fp32")])
def test_chunks(cells, nu, prec):
    s = lattice.generate(*cells, seed=7, check_spd=False)
    seeds = lattice.sample_seeds(s.M, 40, seed=2)
    print(f"[seed chunks M={s.M} nu={nu} {prec}]", flush=True)
    ctx = mar.Context(s.H, s.S)
    try:
        a = ctx.solve(seeds, nu, -0.4, 0.1, precision=prec)
        ctx.set_tuning(upd_q=4)   # the blocks' kernels
        b = ctx.solve(seeds, nu, -0.4, 0.1, precision=prec)
    finally:
        ctx.close()
    assert np.array_equal(a.nu_eff, b.nu_eff)
    tol = 1e-9 if prec == "fp64" else 2e-5
    for x, y in ((a.rho, b.rho), (a.n_seed, b.n_seed), (a.e_seed, b.e_seed)):
        assert np.abs(x - y).max() <= tol * np.abs(y).max()


def test_nearly_exhausted_fp32_regions_run_in_blocks():
    """Regions of fewer than 4 nu rows: the route of the blocks' kernels, bit for bit."""
    s = lattice.generate(6, 5, 5, mixed=True, seed=8, check_spd=False)
    seeds = lattice.sample_seeds(s.M, 50, seed=4)
    ctx = mar.Context(s.H, s.S)
    try:
        ctx.set_local_region(3)
        a = ctx.solve(seeds, 54, -0.4, 0.1, precision="fp32")
        ctx.set_tuning(upd_q=4)   # the blocks' kernels
        b = ctx.solve(seeds, 54, -0.4, 0.1, precision="fp32")
    finally:
        ctx.close()
    assert np.array_equal(a.rho, b.rho) and np.array_equal(a.nu_eff, b.nu_eff)
