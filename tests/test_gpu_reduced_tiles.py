"""The reduced pair system at the edges of its 64-row panels and 64-column
right-hand-side tiles, against the oracle's floating pairs of the assembled
stack.  Both sides are float64 direct solves of systems whose condition stays
below 1e4 at these sizes, so the bar is 1e-10."""
import numpy as np
import pytest

from oracle import reff_oracle as ro
from paper_2607_05818_amd import gen

pytestmark = pytest.mark.gpu


# unknowns (p - 1)(d - 1): 63, 64, 65, 128, 129, 190; endpoints 63, 64, 65, 130
@pytest.mark.parametrize("d,p,m,n", [(2, 64, 30, 33), (2, 65, 31, 33), (2, 66, 32, 33),
                                     (3, 65, 1, 63), (4, 44, 65, 65), (3, 96, 2, 2)])
def test_panel_and_tile_edges(d, p, m, n):
    from paper_2607_05818_amd import reff
    nx, ny = 23, 19
    st = gen.uniform_tier_stack(700 + p, d, 19, p, m, n)
    r_t, s_t = st["r_t"], st["s_t"]
    gx = np.concatenate([np.full(ny * (nx - 1), 1.0 / r) for r in r_t])
    gy = np.concatenate([np.full((ny - 1) * nx, 1.0 / s) for s in s_t])
    desc = gen.make_desc(d, nx, ny, gx, gy, st["tsv_xy"], 1.0 / st["tsv_r"], [[0, 0]])
    ids = lambda xy, t: t * nx * ny + xy[:, 1].astype(np.int64) * nx + xy[:, 0]  # noqa: E731
    want = ro.pairs(desc, ids(st["bump_xy"], 0), ids(st["load_xy"], d - 1), mode=ro.FLOATING)
    print("[case] reduced tiles", d, p, m, n, flush=True)
    got = reff.reff_reduced_pairs(nx, ny, r_t, s_t, st["tsv_xy"], st["tsv_r"], st["bump_xy"],
                                  st["load_xy"])
    assert np.max(np.abs(got - want) / want) <= 1e-10
