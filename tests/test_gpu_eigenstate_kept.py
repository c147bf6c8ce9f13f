"""Eigen states with one workgroup per seed, on the basis that the first pass keeps and (where that would be too large)
on one formed again, against the seed blocks' kernels. The levels agree to rounding (1e-9 of the spectral range, 1e-5 in
FP32); the window around them has slope 1 / sigma, so a component may differ by range / sigma (about 1e3) times that
rounding over the levels' own 1e-10 (FP64): 1e-7 of the largest, 1e-2 in FP32."""
import numpy as np
import pytest

from paper_1307_3218_amd import lattice, mar

pytestmark = pytest.mark.gpu


# 3072 rows at nu = 108: 8.1 GB of basis, formed again
@pytest.mark.parametrize("cells,nu,prec", [((2, 2, 1), 6, "fp64"), ((2, 2, 2), 16, "fp32"), ((4, 3, 3), 30, "fp64"),
                                           ((6, 4, 4), 108, "fp64")])
def test_kept_basis(cells, nu, prec):
    s = lattice.generate(*cells, seed=3, check_spd=False)
    seeds, k = np.arange(s.M), s.M // 2
    print(f"[eigen state kept M={s.M} nu={nu} {prec}]", flush=True)
    ctx = mar.Context(s.H, s.S)
    try:
        a = ctx.eigen_state(seeds, nu, k, 0.05, precision=prec)
        again = ctx.eigen_state(seeds, nu, k, 0.05, precision=prec)
        ctx.set_tuning(upd_q=4)   # the blocks' kernels
        b = ctx.eigen_state(seeds, nu, k, 0.05, precision=prec)
    finally:
        ctx.close()
    assert np.array_equal(a["phi"], again["phi"])
    lo, tol = (1e-9, 1e-7) if prec == "fp64" else (1e-5, 1e-2)
    assert abs(a["eps_k"] - b["eps_k"]) <= lo * 30.0
    x, y = a["phi"], b["phi"]
    y = y if x @ y >= 0 else -y
    assert np.abs(x - y).max() <= tol * np.abs(y).max()
