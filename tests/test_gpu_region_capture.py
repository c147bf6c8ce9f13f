"""Local regions and stream capture: the region is set while the caller's stream captures, and a solve is captured before
the sizes of its regions are known (it runs in seed blocks). Each graph, replayed, gives what an eager call gives."""
import pytest

from paper_1307_3218_amd import lattice, mar

pytestmark = pytest.mark.gpu

NU, SEEDS = 24, 96


def _capture_and_replay(ctx, H, before, want):
    """Captures before() and a solve; each replay, with eager work in between, against the outputs want."""
    import torch
    lst = torch.arange(60, 60 + SEEDS, dtype=torch.int32, device="cuda")
    f = dict(dtype=torch.float64, device="cuda")
    out = dict(d_rho=torch.zeros(H.nnz, **f), d_e_band=torch.zeros(1, **f), d_e_seed=torch.zeros(SEEDS, **f),
               d_n_seed=torch.zeros(SEEDS, **f), d_nu_eff=torch.zeros(SEEDS, dtype=torch.int32, device="cuda"))
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        before()
        ctx.solve_async(lst, NU, -0.3, 0.1, "fp32", **out)
    for _ in range(3):
        for t in out.values():
            t.zero_()
        g.replay()
        torch.cuda.synchronize()
        for k in out:
            assert torch.equal(out[k], want[k]), k


def _eager(ctx, H):
    import torch
    lst = torch.arange(60, 60 + SEEDS, dtype=torch.int32, device="cuda")
    f = dict(dtype=torch.float64, device="cuda")
    out = dict(d_rho=torch.zeros(H.nnz, **f), d_e_band=torch.zeros(1, **f), d_e_seed=torch.zeros(SEEDS, **f),
               d_n_seed=torch.zeros(SEEDS, **f), d_nu_eff=torch.zeros(SEEDS, dtype=torch.int32, device="cuda"))
    ctx.solve_async(lst, NU, -0.3, 0.1, "fp32", **out)
    torch.cuda.synchronize()
    return out


@pytest.fixture(scope="module")
def sysm():
    return lattice.generate(6, 6, 6, mixed=True, seed=3)


def test_region_set_while_the_stream_captures(sysm):
    ctx = mar.Context(sysm.H, sysm.S)
    try:
        ctx.set_local_region(4)
        want = _eager(ctx, sysm.H)
        ctx.set_local_region(6)
        _eager(ctx, sysm.H)
        print("[region set under capture]", flush=True)
        _capture_and_replay(ctx, sysm.H, lambda: ctx.set_local_region(4), want)
    finally:
        ctx.close()


def test_solve_captured_before_the_sizes_are_known(sysm):
    ctx = mar.Context(sysm.H, sysm.S)
    try:
        ctx.set_local_region(4)
        ctx.set_tuning(upd_q=4)     # the blocks' kernels: their workspace is there, the regions are not measured
        want = _eager(ctx, sysm.H)
        ctx.set_tuning()
        print("[solve captured, sizes unknown]", flush=True)
        _capture_and_replay(ctx, sysm.H, lambda: None, want)
    finally:
        ctx.close()
