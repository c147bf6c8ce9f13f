"""The bisections of the device level searches, several halvings to a launch, against the same 200 halvings one at a
time on the host over the levels and weights the device returned: the Fermi level (also at kT = 0, where the count is
a staircase) and, for one seed up to more than one share of the counting workgroups.

The counts differ by the rounding of a sum of 1e3 to 1e5 terms, so the levels agree to 1e-11 of the spectral scale
where the count has slope, and to the width of the step that both fall into at kT = 0.
"""
import numpy as np
import pytest

from oracle import mar_oracle as O
from paper_1307_3218_amd import lattice, mar

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nu,kT,fill", [(1, 1, 0.1, 0.5), (1, 7, 0.0, 1.0), (3, 20, 1e-3, 0.4), (700, 30, 0.1, 1.0),
                                          (700, 30, 0.0, 0.73), (1152, 100, 0.05, 1.3)])
def test_fermi_level_against_host_halvings(n, nu, kT, fill):
    s = lattice.generate(4, 3, 3, mixed=True, seed=8)
    ctx = mar.Context(s.H, s.S)
    try:
        print(f"[level search] {n} seeds nu={nu} kT={kT}", flush=True)
        g, mu = ctx.solve_fermi(np.arange(n), nu, fill * n, kT, levels=True)
    finally:
        ctx.close()
    lo, hi = g.eps.min() - 40 * kT, g.eps.max() + 40 * kT
    for _ in range(200):
        mid = 0.5 * (lo + hi)
        if np.sum(2.0 * O.fermi(g.eps, mid, kT) * g.weight) < fill * n:
            lo = mid
        else:
            hi = mid
    assert abs(mu - 0.5 * (lo + hi)) <= 1e-11 * np.abs(g.eps).max()
    if kT > 0.0:
        assert abs(g.n_seed.sum() - fill * n) <= 1e-10 * n
