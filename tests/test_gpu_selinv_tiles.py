"""Sparse-direct panel kernels at the edges of their tiles: root walls whose
pivot counts sit at and around the 16-column blocks of the tile inverse, the
64-column panels and the 64-row tiles, against the oracle's selected
inversion.  Both sides are float64 without a tolerance; at these sizes (up to
5e3 nodes, fronts of at most a few hundred rows) they differ by rounding of a
few hundred accumulated terms, so the bar is 1e-11."""
import numpy as np
import pytest

from oracle import selinv as osel
from paper_2607_05818_amd import gen

pytestmark = pytest.mark.gpu


# the root's pivots are nt * min(nx, ny) (the wall through every tier)
@pytest.mark.parametrize("nt,nx,ny", [(1, 30, 15), (1, 31, 16), (17, 40, 1), (1, 70, 33), (3, 46, 21),
                                      (2, 67, 32), (5, 29, 13), (3, 47, 42), (3, 45, 43), (4, 36, 48)])
def test_panel_widths(nt, nx, ny):
    from paper_2607_05818_amd import reff
    d = gen.small_random_desc(900 + nt * nx + ny, nt, nx, ny, max(1, nx * ny // 9), 4)
    print("[case] selinv panel widths", nt, nx, ny, flush=True)
    want = osel.diag_full(d)
    h = reff.reff_build_pdn(d)
    got, _ = reff.reff_selinv_diag(h)
    h.close()
    free = want > 0
    assert np.all(got[~free] == 0.0)
    assert np.max(np.abs(got[free] - want[free]) / want[free]) <= 1e-11
