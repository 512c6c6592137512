"""The one-launch Chebyshev application at the edges of its range: stacks of
1023 .. 8193 nodes around its 1024-thread steps and its limits (4096 nodes in
float64, 8192 in float32; the next size up takes the strip passes), thin and
multi-tier ones, and blocks of fewer than 64 columns, against the oracle.
The solver stops at rel_tol 1e-10 (float64) and 1e-5 (mixed) estimated with a
safety factor of four; the estimate is no bound, so the bars are ten times
that, as in the other parity tests."""
import numpy as np
import pytest

from oracle import reff_oracle as ro
from paper_2607_05818_amd import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nt,nx,ny", [(1, 33, 31), (1, 32, 32), (1, 41, 25), (2, 32, 32), (3, 1, 683),
                                      (1, 1365, 3), (4, 32, 32), (1, 17, 241), (2, 64, 64),
                                      (1, 2731, 3)])
def test_sizes(nt, nx, ny):
    from paper_2607_05818_amd import reff
    d = gen.small_random_desc(nt * nx + ny, nt, nx, ny, max(1, nx * ny // 20), 5)
    nodes = gen.sample_free_nodes(d, 70, 3)
    print("[case] resident", nt, nx, ny, flush=True)
    want = ro.diag(d, nodes=nodes)
    h = reff.reff_build_pdn(d)
    got, _ = reff.reff_solve_diag(h, nodes, precision=reff.REFF_PREC_FP64, rel_tol=1e-10)
    assert np.max(np.abs(got - want) / want) <= 1e-9
    got, _ = reff.reff_solve_diag(h, nodes, precision=reff.REFF_PREC_MIXED)
    assert np.max(np.abs(got - want) / want) <= 1e-4
    h.close()


def test_batch_of_small_plans():
    """A batch in which every plan is small, one of them with one tier and no
    TSV; converged blocks leave while others run on."""
    from paper_2607_05818_amd import reff
    plans = [gen.small_random_desc(60 + i, 1 + i % 3, 20 + 3 * i, 37 - 2 * i, 6 if i % 3 else 0, 2 + i)
             for i in range(6)]
    nodes = [gen.sample_free_nodes(d, 10 + 17 * i, i) for i, d in enumerate(plans)]
    print("[case] resident batch", flush=True)
    got, _ = reff.reff_batch_plans(plans, nodes, precision=reff.REFF_PREC_FP64, rel_tol=1e-10)
    for d, v, g in zip(plans, nodes, got):
        want = ro.diag(d, nodes=v)
        assert np.max(np.abs(g - want) / want) <= 1e-9
