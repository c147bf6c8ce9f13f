"""Eigen states on small cells: which way a call takes (the basis of the first pass kept, or formed again), and the same call
under capture, before anything is kept (formed again there: nothing may be allocated) and after. The two ways agree to the
rounding of the levels over the window's width: 1e-7 of the largest component (FP64, sigma = 0.05)."""
import numpy as np
import pytest

from paper_1307_3218_amd import lattice, mar

pytestmark = pytest.mark.gpu

NU, SIGMA = 16, 0.05


@pytest.fixture(scope="module")
def cell():
    return lattice.generate(2, 2, 2, seed=3)


def _call(ctx, M, phi, lv):
    import torch
    st = mar.mar_eigen_state_async(ctx.handle, phi.seeds, M, NU, M // 2, SIGMA, mar.PRECISION["fp64"], mar.FORM["batched"],
                                   phi.t, lv, None, torch.cuda.current_stream().cuda_stream)
    assert st == mar.MAR_OK, mar.mar_last_error(ctx.handle)


class _Phi:
    def __init__(self, M):
        import torch
        self.seeds = torch.arange(M, dtype=torch.int32, device="cuda")
        self.t = torch.zeros(M, dtype=torch.float64, device="cuda")


def _way(ctx, call):
    """'kept' or 'again' (the reference seed solved in the plain form), 'blocks' without k_seed."""
    ctx.profile(True)
    ctx.profile_reset()
    call()
    p = ctx.profile_collect()
    ctx.profile(False)
    if p["dcgs_upd"]["launches"]:
        return "blocks"
    return "again" if p["cgs_proj_KSK"]["launches"] + p["cgs_proj_1"]["launches"] else "kept"


def _close(a, b):
    a, b = a.cpu().numpy(), b.cpu().numpy()
    b = b if a @ b >= 0 else -b
    assert np.abs(a - b).max() <= 1e-7 * np.abs(b).max()


def test_ways(cell):
    ctx = mar.Context(cell.H, cell.S)
    try:
        seeds = np.arange(cell.M)
        assert _way(ctx, lambda: ctx.eigen_state(seeds, NU, cell.M // 2, SIGMA)) == "kept"
        ctx.set_tuning(upd_q=4)
        assert _way(ctx, lambda: ctx.eigen_state(seeds, NU, cell.M // 2, SIGMA)) == "blocks"
    finally:
        ctx.close()
    s = lattice.generate(6, 4, 4, seed=3, check_spd=False)
    ctx = mar.Context(s.H, s.S)
    try:   # 8.1 GB of basis
        assert _way(ctx, lambda: ctx.eigen_state(np.arange(s.M), 108, s.M // 2, SIGMA)) == "again"
    finally:
        ctx.close()


@pytest.mark.parametrize("kept", [False, True])
def test_under_capture(cell, kept):
    import torch
    M = cell.M
    want, got = _Phi(M), _Phi(M)
    lv = torch.zeros(3, dtype=torch.float64, device="cuda")
    other = mar.Context(cell.H, cell.S)
    try:
        _call(other, M, want, lv)
        torch.cuda.synchronize()
    finally:
        other.close()
    levels = lv.clone()
    ctx = mar.Context(cell.H, cell.S)
    try:
        if not kept:
            ctx.set_tuning(upd_q=4)   # the blocks' workspaces are there, nothing is kept
        _call(ctx, M, got, lv)
        ctx.set_tuning()
        torch.cuda.synchronize()
        print(f"[eigen state under capture, kept before: {kept}]", flush=True)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            _call(ctx, M, got, lv)
        for _ in range(3):
            got.t.zero_()
            lv.zero_()
            g.replay()
            torch.cuda.synchronize()
            assert (lv - levels).abs().max().item() <= 1e-9 * 30.0
            _close(got.t, want.t)
    finally:
        ctx.close()
