"""FP64 local regions that run in seed blocks: five to eight seeds take a block of 16 up to 16 hops (blocks of 8 are a fifth
to a third slower there), fewer seeds and deeper regions the least power of two. Widths differ in the partition of their
sums, so the default gives the bits of the width that it takes."""
import numpy as np
import pytest

from paper_1307_3218_amd import lattice, mar

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hops,seeds,width", [(10, 8, 16), (12, 5, 16), (16, 8, 16), (17, 8, 8), (10, 4, 4), (10, 9, 16)])
def test_width(hops, seeds, width):
    s = lattice.generate(14, 14, 14, mixed=True, seed=1, check_spd=False)
    lst = np.arange(s.M // 2, s.M // 2 + seeds, dtype=np.int32)
    out = {}
    ctx = mar.Context(s.H, s.S)
    try:
        ctx.set_local_region(hops)
        for b in (0, 4, 8, 16):
            if b == 4 and seeds > 4:
                continue
            ctx.set_tuning(seed_block=b)
            out[b] = ctx.solve(lst, 40, -0.4, 0.1, precision="fp64").rho
    finally:
        ctx.close()
    same = [b for b in out if b and np.array_equal(out[b], out[0])]
    print(f"[width] {hops} hops {seeds} seeds: equal to {same}", flush=True)
    assert same == [width]
