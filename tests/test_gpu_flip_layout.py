"""The flipping's work layout at its edges against the flip oracle, whose decisions it must take exactly: one colour for
all rows (a diagonal pair) in one and in several rounds of the workgroup, rows longer than the entries kept in
registers, and the residual in LDS or, past the rows that fit there, in memory."""
import numpy as np
import pytest
import scipy.sparse as sp

from oracle import mar_flip as OF
from paper_1307_3218_amd import lattice, mar

pytestmark = pytest.mark.gpu


def _diagonal(n):
    rng = np.random.default_rng(n)
    return sp.diags(rng.standard_normal(n)).tocsr(), sp.identity(n, format="csr")


def _long_rows(n, k):
    """A symmetric pair whose rows store up to 2 k + 1 entries (cyclic neighbours i +- d, d <= k, one row less)."""
    rng = np.random.default_rng(n + k)
    i = np.arange(n)
    r = np.concatenate([i[i != 5] for _ in range(k)] + [i])
    c = np.concatenate([(i[i != 5] + d) % n for d in range(1, k + 1)] + [i])
    H = sp.coo_matrix((rng.standard_normal(len(r)), (r, c)), shape=(n, n))
    H = (H + H.T).tocsr()
    S = H.copy()
    S.data = np.where(np.repeat(i, np.diff(H.indptr)) == H.indices, 1.0, 0.5 / (4 * k))
    return H, S


CASES = {"one_row": lambda: _diagonal(1), "one_colour": lambda: _diagonal(500), "one_colour_rounds": lambda: _diagonal(1700),
         "rows_of_21": lambda: _long_rows(300, 10), "rows_of_63": lambda: _long_rows(1500, 31),
         "residual_in_memory": lambda: (lambda s: (s.H.tocsr(), s.S.tocsr()))(
             lattice.generate(9, 8, 8, mixed=True, seed=2, check_spd=False))}


@pytest.mark.parametrize("penalty", [False, True])
@pytest.mark.parametrize("name", sorted(CASES))
def test_layout_edges(name, penalty):
    H, S = CASES[name]()
    M = H.shape[0]
    rng = np.random.default_rng(3)
    x, ref = rng.standard_normal(M), (rng.standard_normal(M) if penalty else None)
    c = 50.0 * OF.C_PAPER_EV2 if penalty else 0.0
    want = OF.local_flip(H, S, x, 0.3, phi_ref=ref, c=c, max_sweeps=4)
    print(f"[flip {name} M={M} penalty={penalty}] rows to {np.diff(H.indptr).max()} flips {want.flips}", flush=True)
    ctx = mar.Context(H, S)
    try:
        got = ctx.local_flip(x, 0.3, phi_ref=ref, c=c, max_sweeps=4)
    finally:
        ctx.close()
    assert got["sweeps"] == want.sweeps and got["flips"] == want.flips
    assert np.array_equal(got["phi"], want.phi)
    np.testing.assert_allclose(got["R"], want.R, rtol=1e-10)
