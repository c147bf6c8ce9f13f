"""One workgroup per seed in chunks that a bounded workspace shortens: the static scratch of mar_solve_async_noalloc, and
the context's own under capture, where it cannot grow. A seed's results do not depend on its chunk, so they equal those of
an unbounded call bit for bit (which the seed blocks' would not)."""
import numpy as np
import pytest

from paper_1307_3218_amd import lattice, mar

pytestmark = pytest.mark.gpu


def _buffers(H, n):
    import torch
    f = dict(dtype=torch.float64, device="cuda")
    return dict(d_rho=torch.zeros(H.nnz, **f), d_e_band=torch.zeros(1, **f), d_e_seed=torch.zeros(n, **f),
                d_n_seed=torch.zeros(n, **f), d_nu_eff=torch.zeros(n, dtype=torch.int32, device="cuda"))


def _seedwise(ctx, call):
    """Whether call's solve ran k_seed: no products or updates of the blocks' schedule, one launch of the seed form."""
    ctx.profile(True)
    ctx.profile_reset()
    call()
    p = ctx.profile_collect()
    ctx.profile(False)
    return p["spmm"]["launches"] == p["dcgs_upd"]["launches"] == 0 and p["cgs_upd"]["launches"] > 0


# 1024 rows, FP64, nu = 100: the basis of 90 workgroups takes 61 of the scratch's 67 MB, the subspace matrices 94 KB a seed
@pytest.mark.parametrize("seeds", [90, 61])
def test_static_scratch(seeds):
    import torch
    s = lattice.generate(4, 4, 2, seed=1)
    lst = torch.arange(17, 17 + seeds, dtype=torch.int32, device="cuda")
    a, b = _buffers(s.H, seeds), _buffers(s.H, seeds)
    ctx = mar.Context(s.H, s.S)
    try:
        assert _seedwise(ctx, lambda: ctx.solve_async(lst, 100, -0.4, 0.1, "fp64", **a))
        print(f"[short chunks, static scratch: {seeds} seeds]", flush=True)
        st = mar.mar_solve_async_noalloc(ctx.handle, lst, seeds, 100, -0.4, 0.1, mar.PRECISION["fp64"],
                                         mar.FORM["batched"], b["d_rho"], b["d_e_band"], b["d_e_seed"], b["d_n_seed"],
                                         b["d_nu_eff"], stream=torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
    finally:
        ctx.close()
    assert st == mar.MAR_OK
    for k in a:
        assert torch.equal(a[k], b[k]), k


@pytest.mark.parametrize("nu,prec", [(12, "fp32"), (60, "fp64")])
def test_more_seeds_captured_than_warmed(nu, prec):
    import torch
    s = lattice.generate(4, 4, 2, seed=1)
    lst = torch.arange(s.M, dtype=torch.int32, device="cuda")
    want, out = _buffers(s.H, s.M), _buffers(s.H, s.M)
    other = mar.Context(s.H, s.S)
    try:
        assert _seedwise(other, lambda: other.solve_async(lst, nu, -0.4, 0.1, prec, **want))
    finally:
        other.close()
    ctx = mar.Context(s.H, s.S)
    try:
        ctx.solve_async(lst[:300], nu, -0.4, 0.1, prec, **_buffers(s.H, 300))
        torch.cuda.synchronize()
        print(f"[short chunks under capture: nu={nu} {prec}]", flush=True)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            ctx.solve_async(lst, nu, -0.4, 0.1, prec, **out)
        for _ in range(3):
            for t in out.values():
                t.zero_()
            g.replay()
            torch.cuda.synchronize()
            for k in out:
                assert torch.equal(out[k], want[k]), k
    finally:
        ctx.close()


# the basis of FP64 nu = 60 on 1024 rows does not fit in LDS: 200 workgroups need more memory than 130 of the warm call
@pytest.mark.parametrize("warm,seeds", [(130, 200), (100, 512)])
def test_fewer_workgroups_under_capture(warm, seeds):
    import torch
    s = lattice.generate(4, 4, 2, seed=1)
    lst = torch.arange(seeds, dtype=torch.int32, device="cuda")
    want, out = _buffers(s.H, seeds), _buffers(s.H, seeds)
    other = mar.Context(s.H, s.S)
    try:
        assert _seedwise(other, lambda: other.solve_async(lst, 60, -0.4, 0.1, "fp64", **want))
    finally:
        other.close()
    ctx = mar.Context(s.H, s.S)
    try:
        ctx.solve_async(lst[:warm], 60, -0.4, 0.1, "fp64", **_buffers(s.H, warm))
        torch.cuda.synchronize()
        print(f"[fewer workgroups under capture: {warm}, {seeds}]", flush=True)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            ctx.solve_async(lst, 60, -0.4, 0.1, "fp64", **out)
        for _ in range(3):
            for t in out.values():
                t.zero_()
            g.replay()
            torch.cuda.synchronize()
            for k in out:
                assert torch.equal(out[k], want[k]), k
    finally:
        ctx.close()
