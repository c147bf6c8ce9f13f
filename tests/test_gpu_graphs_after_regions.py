"""mar_solve_many on contexts whose earlier solves ran one workgroup per seed in local regions of six hops and more: no two
seed blocks were in flight there, so nothing refuses the context, and the graph gives what an eager call gives."""
import numpy as np
import pytest

from paper_1307_3218_amd import lattice, mar

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hops,seeds", [(6, 300), (8, 513)])   # more seeds than the widest block
def test_solve_many_after_seedwise_regions(hops, seeds):
    import torch
    s = lattice.generate(6, 6, 6, mixed=True, seed=3)
    lst = torch.arange(40, 40 + seeds, dtype=torch.int32, device="cuda")

    def buffers():
        f = dict(dtype=torch.float64, device="cuda")
        return dict(d_rho=torch.zeros(s.H.nnz, **f), d_e_band=torch.zeros(1, **f), d_e_seed=torch.zeros(seeds, **f),
                    d_nu_eff=torch.zeros(seeds, dtype=torch.int32, device="cuda"))

    c = mar.Context(s.H, s.S)
    try:
        c.set_local_region(hops)
        c.profile(True)
        eager, many = buffers(), buffers()
        c.solve_async(lst, 24, -0.3, 0.1, "fp32", **eager)
        p = c.profile_collect()
        c.profile(False)
        assert p["spmm"]["launches"] == p["dcgs_upd"]["launches"] == 0 and p["cgs_upd"]["launches"] > 0   # k_seed ran
        c.solve_async(lst, 24, -0.3, 0.1, "fp32", **eager)
        print(f"[graph after regions of {hops} hops]", flush=True)
        for _ in range(3):
            mar.solve_many([c], [dict(d_seeds=lst, nu=24, mu=-0.3, kT=0.1, precision="fp32", **many)])
            torch.cuda.synchronize()
            for k in eager:
                assert torch.equal(eager[k], many[k]), k
    finally:
        c.close()
