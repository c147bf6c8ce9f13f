"""Which kernels a batched solve runs, on either side of the lines: one workgroup per seed, or seed blocks (few seeds on
many rows, where one compute unit per seed is slower). The profile tells: the seed form launches no products."""
import numpy as np
import pytest

from paper_1307_3218_amd import lattice, mar

pytestmark = pytest.mark.gpu


def _route(ctx, seeds, nu, prec):
    ctx.profile(True)
    ctx.profile_reset()
    out = ctx.solve(seeds, nu, -0.4, 0.1, precision=prec)
    p = ctx.profile_collect()
    ctx.profile(False)
    assert np.all(out.nu_eff == nu)
    return "seeds" if p["spmm"]["launches"] == 0 and p["cgs_upd"]["launches"] > 0 else "blocks"


@pytest.mark.parametrize("cells,prec,nu,seeds,want", [
    ((2, 2, 2), "fp32", 30, 1, "seeds"), ((6, 4, 4), "fp64", 100, 1, "seeds"), ((6, 4, 4), "fp32", 120, 300, "seeds"),
    ((8, 4, 4), "fp32", 60, 4, "seeds"), ((8, 4, 4), "fp32", 64, 4, "blocks"), ((8, 4, 4), "fp64", 42, 2, "seeds"),
    ((8, 4, 4), "fp64", 64, 1, "blocks"), ((8, 4, 4), "fp64", 100, 2, "blocks"), ((7, 4, 4), "fp64", 100, 128, "blocks"),
    ((8, 4, 4), "fp64", 100, 129, "seeds"), ((8, 4, 4), "fp64", 130, 200, "blocks"), ((9, 4, 4), "fp32", 12, 200, "blocks")])
def test_whole_cells(cells, prec, nu, seeds, want):
    s = lattice.generate(*cells, seed=1, check_spd=False)
    ctx = mar.Context(s.H, s.S)
    try:
        assert _route(ctx, np.arange(8, 8 + seeds, dtype=np.int32), nu, prec) == want
    finally:
        ctx.close()


@pytest.fixture(scope="module")
def regions():
    s = lattice.generate(14, 14, 14, mixed=True, seed=1, check_spd=False)
    ctx = mar.Context(s.H, s.S)
    yield s, ctx
    ctx.close()


# mixed lattice: the largest regions of 9, 10, 11 and 12 hops have 2768, 3720, 4888 and 6284 rows
@pytest.mark.parametrize("hops,prec,nu,seeds,want", [
    (9, "fp64", 40, 2, "seeds"), (10, "fp32", 40, 4, "seeds"), (10, "fp32", 31, 4, "blocks"), (11, "fp32", 40, 4, "seeds"),
    (12, "fp32", 40, 64, "blocks"), (12, "fp32", 40, 65, "seeds"), (12, "fp32", 100, 16, "blocks"),
    (10, "fp64", 40, 32, "blocks"), (10, "fp64", 40, 33, "seeds"), (12, "fp64", 40, 200, "blocks"),
    (80, "fp32", 12, 4, "blocks")])
def test_local_regions(regions, hops, prec, nu, seeds, want):
    s, ctx = regions
    ctx.set_local_region(hops)
    assert _route(ctx, np.arange(s.M // 2, s.M // 2 + seeds, dtype=np.int32), nu, prec) == want


def test_fp32_regions_on_either_side_of_a_quarter_of_the_rows(regions):
    """3 hops, regions of 19 to 41 block rows: up to nu = 41 one workgroup per seed (regions with fewer than 4 nu rows among
    them), above that the blocks."""
    s, ctx = regions
    ctx.set_local_region(3)
    lst = np.arange(s.M // 2, s.M // 2 + 40, dtype=np.int32)
    assert _route(ctx, lst, 41, "fp32") == "seeds" and _route(ctx, lst, 41, "fp64") == "seeds"
    assert _route(ctx, lst, 42, "fp32") == "blocks" and _route(ctx, lst, 42, "fp64") == "seeds"


def test_profiled_bytes_are_operands_and_results_once():
    """256 rows, nu = 30, FP32: the blocks of H and S with their columns, the subspace matrices and the gathered rows."""
    s = lattice.generate(2, 2, 2, seed=0)
    ctx = mar.Context(s.H, s.S)
    try:
        ctx.profile(True)
        ctx.solve(np.arange(256, dtype=np.int32), 30, -0.4, 0.1, precision="fp32")
        p = ctx.profile_collect()["cgs_upd"]
    finally:
        ctx.close()
    blocks, row = s.H.nnz // 16, int(np.diff(s.H.tocsr().indptr).max())
    assert p["launches"] == 1
    assert p["bytes"] == blocks * (2 * 16 * 4 + 4) + 64 * 4 + 256 * 30 * (31 / 2 + row) * 8
