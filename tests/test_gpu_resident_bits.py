"""The one-launch Chebyshev application gives the bits of the strip passes.  A
launch group takes it only if every stack of it is small, so the same small plan
alone and beside a larger one goes both ways; its work units, their reductions and
its columns are the same in both calls (up to 512 chunks of 32 nodes a plan, a
unit each), so every bit of its results has to be.  Tiers of one row have the
same strips whatever their height, which float32 needs: its strips carry the
partial Grams."""
import numpy as np
import pytest

from paper_2607_05818_amd import gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,small,large", [("fp64", (2, 32, 32), (2, 64, 65)), ("fp64", (1, 61, 47), (3, 50, 41)),
                                              ("fp64", (4, 1, 700), (1, 4200, 1)),
                                              ("mixed", (2, 1500, 1), (3, 3000, 1)),
                                              ("mixed", (4, 2000, 1), (2, 4200, 1))])
@pytest.mark.parametrize("degree", [2, 3, 4, 19, 20])
def test_same_bits_as_strip_passes(prec, small, large, degree):
    from paper_2607_05818_amd import reff
    p = reff.REFF_PREC_FP64 if prec == "fp64" else reff.REFF_PREC_MIXED
    mk = lambda s, seed: gen.small_random_desc(seed, *s, max(1, s[1] * s[2] // 15) if s[0] > 1 else 0,  # noqa: E731
                                               max(8, s[1] * s[2] // 40))
    a, b = mk(small, 4), mk(large, 5)
    limit = 4096 if prec == "fp64" else 8192
    assert gen.n_nodes(a) <= limit < gen.n_nodes(b)
    na, nb = gen.sample_free_nodes(a, 60, 1), gen.sample_free_nodes(b, 60, 2)
    print("[case] resident bits", prec, small, large, degree, flush=True)
    alone, _ = reff.reff_batch_plans([a], [na], precision=p, precond_degree=degree)
    both, _ = reff.reff_batch_plans([a, b], [na, nb], precision=p, precond_degree=degree)
    assert np.array_equal(alone[0], both[0])
