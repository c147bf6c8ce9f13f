"""The autotuner where solves run one workgroup per seed: what it reports is what later solves do. On a cell of 256 rows
that form is several times faster than any seed block, so a rate that belongs to the blocks is off by that factor."""
import time

import numpy as np
import pytest

from paper_1307_3218_amd import lattice, mar

pytestmark = pytest.mark.gpu


def test_reported_rate_is_that_of_later_solves():
    import torch
    s = lattice.generate(2, 2, 2, seed=0)
    seeds = torch.arange(256, dtype=torch.int32, device="cuda")
    f = dict(dtype=torch.float64, device="cuda")
    out = dict(d_rho=torch.zeros(s.H.nnz, **f), d_e_band=torch.zeros(1, **f))
    ctx = mar.Context(s.H, s.S)
    try:
        t = ctx.autotune(seeds, 30, -0.3, 0.1, "fp32")

        def rate():
            best = 0.0
            for _ in range(8):
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                ctx.solve_async(seeds, 30, -0.3, 0.1, "fp32", **out)
                torch.cuda.synchronize()
                best = max(best, 256 / (time.perf_counter() - t0))
            return best

        later = rate()
        ctx.set_tuning(seed_block=t["seed_block"], proj_variant=t["proj_variant"])   # the reported block itself
        blocks = rate()
    finally:
        ctx.close()
    print(f"[autotune] {t}; later solves {later:.0f}/s, in the reported block {blocks:.0f}/s", flush=True)
    assert later >= 2.0 * blocks
    assert 0.5 * later <= t["probe_rate"] <= 2.0 * later
    assert t["seed_block"] in (16, 32, 64, 128, 256) and t["proj_variant"] in (0, 3)
