"""Seed counts that fill no block: the last, narrower blocks of a solve against the same seeds in blocks of one pinned
width, on a 4x4-block and on a general CSR system (with rows that are padded to a multiple of four), and a solve whose
seeds all lie in narrower blocks. The two differ in the partition of their sums only: 1e-9 (FP64) and 2e-5 (FP32) of the
largest value."""
import numpy as np
import pytest

from paper_1307_3218_amd import lattice, mar

pytestmark = pytest.mark.gpu

# cells, rows cut, precision, nu, seeds: 128 + 1, 128 + 44 (CSR), 256 + 128, 256 + 33, 64 + 16 (70 seeds, wide sweeps), 5
CASES = [((8, 8, 4), 0, "fp64", 20, 129), ((8, 8, 4), 3, "fp64", 20, 172), ((8, 8, 4), 0, "fp32", 30, 384),
         ((8, 8, 4), 1, "fp32", 25, 289), ((8, 8, 8), 0, "fp64", 100, 70), ((8, 8, 4), 0, "fp64", 9, 5)]


@pytest.mark.parametrize("cells,cut,prec,nu,n", CASES)
def test_widths_agree(cells, cut, prec, nu, n):
    s = lattice.generate(*cells, seed=4, check_spd=False)
    M = s.M - cut
    H, S = s.H[:M, :M].tocsr(), s.S[:M, :M].tocsr()
    seeds = lattice.sample_seeds(M, n, seed=n)
    ctx = mar.Context(H, S)
    try:
        print(f"[block widths M={M} {prec} nu={nu} n={n}]", flush=True)
        a = ctx.solve(seeds, nu, -0.4, 0.1, precision=prec, levels=True)
        ctx.set_tuning(seed_block=64)
        b = ctx.solve(seeds, nu, -0.4, 0.1, precision=prec, levels=True)
    finally:
        ctx.close()
    tol = 1e-9 if prec == "fp64" else 2e-5
    assert np.array_equal(a.nu_eff, b.nu_eff)
    for x, y in ((a.rho, b.rho), (a.e_seed, b.e_seed), (a.n_seed, b.n_seed)):
        assert np.abs(x - y).max() <= tol * np.abs(y).max()
