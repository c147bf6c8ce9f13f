"""The support search of few levels on many rows, with seeds all over the cell: the levels are launches there (one workgroup
would walk every row: 232 us whatever the levels). The search of nu = 2 takes well under that of nu = 100, and the solve
gives what the one without support tracking gives (FP64, 1e-9 of the largest)."""
import numpy as np
import pytest

from paper_1307_3218_amd import lattice, mar

pytestmark = pytest.mark.gpu


def test_few_levels_on_many_rows():
    import torch
    s = lattice.generate(16, 16, 16, mixed=True, seed=1, check_spd=False)
    f = dict(dtype=torch.float64, device="cuda")
    out = dict(d_rho=torch.zeros(s.H.nnz, **f), d_e_band=torch.zeros(1, **f))
    lst = lattice.sample_seeds(s.M, 256, seed=2).astype(np.int32)
    d_lst = torch.from_numpy(lst).cuda()
    ctx = mar.Context(s.H, s.S)
    try:
        ms = {}
        for nu in (2, 100):
            for _ in range(4):
                ctx.profile(True)
                ctx.profile_reset()
                ctx.solve_async(d_lst, nu, -0.4, 0.1, "fp32", **out)
                torch.cuda.synchronize()
                ms[nu] = min(ms.get(nu, 1e9), ctx.profile_collect()["support"]["ms"])
                ctx.profile(False)
        print(f"[support] search of nu = 2 {ms[2] * 1e3:.0f} us, nu = 100 {ms[100] * 1e3:.0f} us", flush=True)
        got = []
        for support in (True, False):
            ctx.set_tuning(seed_block=64, support=support)
            got.append(ctx.solve(lst, 6, -0.4, 0.1, precision="fp64"))
    finally:
        ctx.close()
    a, b = got
    assert np.array_equal(a.nu_eff, b.nu_eff)
    for x, y in ((a.rho, b.rho), (a.e_seed, b.e_seed), (a.n_seed, b.n_seed)):
        assert np.abs(x - y).max() <= 1e-9 * np.abs(y).max()
    assert ms[2] <= 0.6 * ms[100]
