"""Strip heights by rounds: tiers whose rows leave ragged last segments, one
segment, one-row strips, and a batch of different stacks, both precisions,
against the oracle.  rel_tol 1e-10 (float64) and 1e-5 (mixed) are estimates,
not bounds: the bars are ten times that, as in the other parity tests."""
import numpy as np
import pytest

from oracle import reff_oracle as ro
from paper_2607_05818_amd import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nt,nx,ny", [(2, 70, 63), (2, 70, 65), (1, 140, 127), (1, 33, 300),
                                      (1, 300, 33), (1, 8200, 1), (3, 97, 128)])
def test_heights(nt, nx, ny):
    from paper_2607_05818_amd import reff
    d = gen.small_random_desc(nx, nt, nx, ny, 30 if nt > 1 else 0, max(5, nx // 20))
    nodes = gen.sample_free_nodes(d, 20, 3)
    print("[case] strips", nt, nx, ny, flush=True)
    want = ro.diag(d, nodes=nodes)
    h = reff.reff_build_pdn(d)
    got, _ = reff.reff_solve_diag(h, nodes, precision=reff.REFF_PREC_FP64, rel_tol=1e-10)
    assert np.max(np.abs(got - want) / want) <= 1e-9
    got, _ = reff.reff_solve_diag(h, nodes, precision=reff.REFF_PREC_MIXED)
    assert np.max(np.abs(got - want) / want) <= 1e-4
    h.close()


def test_batch_of_unequal_stacks():
    from paper_2607_05818_amd import reff
    plans = [gen.small_random_desc(80 + i, 1 + i % 3, 30 + 17 * i, 130 - 13 * i, 10 if i % 3 else 0, 5)
             for i in range(8)]
    nodes = [gen.sample_free_nodes(d, 16, i) for i, d in enumerate(plans)]
    print("[case] strips batch", flush=True)
    got, _ = reff.reff_batch_plans(plans, nodes, precision=reff.REFF_PREC_MIXED)
    for d, v, g in zip(plans, nodes, got):
        want = ro.diag(d, nodes=v)
        assert np.max(np.abs(g - want) / want) <= 1e-4
