"""Float64 three-step Chebyshev passes (stacks above the one-launch limit):
strip widths around the 32-node tile, ragged last segments, tiers joined by TSV
columns at every edge, and degrees that leave remainders of two and one steps,
against the oracle.  The solver stops at an estimated 2.5e-11 relative; the
estimate is no bound, so the bar is 1e-9."""
import numpy as np
import pytest

from oracle import reff_oracle as ro
from paper_2607_05818_amd import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nt,nx,ny,degree", [(2, 65, 33, 4), (2, 31, 90, 5), (3, 97, 40, 6),
                                             (1, 129, 70, 19), (4, 32, 35, 20), (2, 33, 64, 32)])
def test_fp64_passes(nt, nx, ny, degree):
    from paper_2607_05818_amd import reff
    d = gen.small_random_desc(nx + ny, nt, nx, ny, nx * ny // 12, 6)
    if nt > 1:  # TSVs in all four corners as well
        corner = np.array([[0, 0], [nx - 1, 0], [0, ny - 1], [nx - 1, ny - 1]], dtype=np.int32)
        keep = [k for k, v in enumerate(d["tsv_xy"]) if not any((v == c).all() for c in corner)]
        d["tsv_xy"] = np.concatenate([d["tsv_xy"][keep], corner])
        d["tsv_g"] = np.concatenate([d["tsv_g"][keep], np.full((4, nt - 1), 3.0)])
    nodes = gen.sample_free_nodes(d, 80, 9)
    print("[case] cheb3 fp64", nt, nx, ny, degree, flush=True)
    want = ro.diag(d, nodes=nodes)
    h = reff.reff_build_pdn(d)
    got, _ = reff.reff_solve_diag(h, nodes, precision=reff.REFF_PREC_FP64, rel_tol=1e-10,
                                  precond_degree=degree)
    h.close()
    assert np.max(np.abs(got - want) / want) <= 1e-9
