"""The guarded 64 x 64 inversions of the block solver where columns drop out:
blocks of 1 .. 64 columns around the 16-column steps (the empty columns have
zero pivots), and a stack just large enough for the block method, solved so
far that its block residual loses column rank, against the oracle.  The solver
stops at rel_tol 1e-11 (float64) and 1e-5 (mixed), estimated with a safety
factor of four; the estimate is no bound and the oracle's own rounding is of
the order 1e-11, so the bars are 1e-9 and ten times 1e-5."""
import numpy as np
import pytest

from oracle import reff_oracle as ro
from paper_2607_05818_amd import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count", [1, 2, 15, 16, 17, 31, 33, 48, 49, 63, 64])
def test_columns(count):
    from paper_2607_05818_amd import reff
    d = gen.small_random_desc(7, 2, 29, 23, 40, 6)
    nodes = gen.sample_free_nodes(d, count, count)
    print("[case] small matrices", count, flush=True)
    want = ro.diag(d, nodes=nodes)
    h = reff.reff_build_pdn(d)
    got, _ = reff.reff_solve_diag(h, nodes, precision=reff.REFF_PREC_FP64, rel_tol=1e-11)
    assert np.max(np.abs(got - want) / want) <= 1e-9
    got, _ = reff.reff_solve_diag(h, nodes, precision=reff.REFF_PREC_MIXED)
    assert np.max(np.abs(got - want) / want) <= 1e-4
    h.close()


@pytest.mark.parametrize("degree", [8, 0])
def test_rank_loss(degree):
    """Neighbouring columns, the nearest to dependent ones."""
    from paper_2607_05818_amd import reff
    d = gen.small_random_desc(11, 1, 41, 26, 0, 8)
    free = np.setdiff1d(np.arange(gen.n_nodes(d)), gen.pad_ids(d))[:64]
    print("[case] rank loss", degree, flush=True)
    want = ro.diag(d, nodes=free)
    h = reff.reff_build_pdn(d)
    got, st = reff.reff_solve_diag(h, free, precision=reff.REFF_PREC_FP64, rel_tol=1e-11,
                                   precond_degree=degree)
    print("  iterations", st["iters_total"], flush=True)
    assert np.max(np.abs(got - want) / want) <= 1e-9
    h.close()
