"""Sums of the partial Gram matrices over a block's units, four or sixteen
waves side by side: stacks of 63 .. 193 units of 32 nodes around the change
at 64 units and the waves' remainders, one and two solve blocks, against the
oracle.  rel_tol 1e-10 is an estimate, not a bound: the bar is ten times
that, as in the other parity tests."""
import numpy as np
import pytest

from oracle import reff_oracle as ro
from paper_2607_05818_amd import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx", [63, 64, 65, 67, 111, 113, 128, 193])
def test_units(nx):
    from paper_2607_05818_amd import reff
    d = gen.small_random_desc(nx, 1, nx, 32, 0, 5)
    nodes = gen.sample_free_nodes(d, 64 if nx % 2 else 70, 3)
    print("[case] reduce", nx, flush=True)
    want = ro.diag(d, nodes=nodes)
    h = reff.reff_build_pdn(d)
    got, _ = reff.reff_solve_diag(h, nodes, precision=reff.REFF_PREC_FP64, rel_tol=1e-10)
    assert np.max(np.abs(got - want) / want) <= 1e-9
    h.close()
