"""Seeds that fill no block: one padded block, or two narrower ones where that saves more than it costs (FP64 later than
FP32). Widths differ in the partition of their sums, so the first seeds' bits tell the width that they ran in."""
import numpy as np
import pytest

from paper_1307_3218_amd import lattice, mar

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cells,prec,nu,seeds,width", [
    ((8, 8, 8), "fp64", 100, 70, 128), ((8, 8, 16), "fp64", 80, 70, 64), ((8, 8, 8), "fp64", 100, 40, 64),
    ((8, 8, 8), "fp32", 100, 140, 128), ((8, 8, 8), "fp32", 60, 140, 128), ((8, 8, 8), "fp32", 40, 140, 256)])
def test_first_block(cells, prec, nu, seeds, width):
    s = lattice.generate(*cells, seed=1, check_spd=False)
    lst = lattice.sample_seeds(s.M, seeds, seed=5).astype(np.int32)
    out = {}
    ctx = mar.Context(s.H, s.S)
    try:
        for b in (0, width // 2, width, width * 2):
            if b > (128 if prec == "fp64" else 256):
                continue
            ctx.set_tuning(seed_block=b)
            out[b] = ctx.solve(lst, nu, -0.4, 0.1, precision=prec).e_seed[:16]
    finally:
        ctx.close()
    same = [b for b in out if b and np.array_equal(out[b], out[0])]
    print(f"[split] {s.M} rows {prec} nu={nu} {seeds} seeds: first block {same}", flush=True)
    assert same == [width]
