"""General CSR products where a row's entries are not a multiple of the eight in flight: the remainder costs no more than its
entries. Per entry, rows of 31 (three eights and seven) take at most half as long again as rows of 63 (seven eights and
seven), in FP32 with blocks of 256 seeds, where a row is a wavefront."""
import numpy as np
import pytest
import scipy.sparse as sp

from paper_1307_3218_amd import mar

pytestmark = pytest.mark.gpu


def test_time_per_entry():
    import torch
    f = dict(dtype=torch.float64, device="cuda")
    per_entry = {}
    for n, half in ((20001, 15), (12001, 31)):
        H = sp.diags([np.full(n - abs(k), 1.0 / (1 + abs(k))) for k in range(-half, half + 1)],
                     range(-half, half + 1)).tocsr()
        lst = torch.arange(n // 2, n // 2 + 256, dtype=torch.int32, device="cuda")
        out = dict(d_rho=torch.zeros(H.nnz, **f), d_e_band=torch.zeros(1, **f))
        ctx = mar.Context(H, sp.eye(n).tocsr())
        try:
            best = 1e9
            for _ in range(5):
                ctx.profile(True)
                ctx.profile_reset()
                ctx.solve_async(lst, 30, -0.4, 0.1, "fp32", **out)
                torch.cuda.synchronize()
                best = min(best, ctx.profile_collect()["spmm"]["ms"])
                ctx.profile(False)
        finally:
            ctx.close()
        per_entry[half] = best / (n * (2 * half + 1))
    print(f"[csr] per entry, rows of 31 / of 63: {per_entry[15] / per_entry[31]:.2f}", flush=True)
    assert per_entry[15] <= 1.5 * per_entry[31]
