"""The reduced pair system of a stack of more tiers than one launch of the table
products takes (65535, their grid's z): 2 x 2 tiers joined by one TSV column,
whose pairs are sums in closed form, R = R_0(bump, TSV) + the TSV's segments +
R_last(TSV, load).  The sum of 66,000 positive terms in float64 is off by at most
66,000 eps = 1.5e-11; the bar is 1e-10."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_more_tiers_than_a_launch():
    from paper_2607_05818_amd import reff
    d = 66000
    rng = np.random.default_rng(6)
    r, s = rng.uniform(0.5, 2, d), rng.uniform(0.5, 2, d)
    tr = rng.uniform(0.5, 2, (1, d - 1))
    ring = lambda a, b: a * (a + 2 * b) / (2 * a + 2 * b)  # noqa: E731  neighbours along the a edges
    bump = np.array([[0, 0], [1, 0]], dtype=np.int32)
    load = np.array([[0, 0], [0, 1]], dtype=np.int32)
    want = np.array([0.0, ring(r[0], s[0])])[:, None] + np.array([0.0, ring(s[-1], r[-1])])[None, :] + tr.sum()
    print("[case] reduced many tiers", flush=True)
    got = reff.reff_reduced_pairs(2, 2, r, s, np.array([[0, 0]], dtype=np.int32), tr, bump, load)
    assert np.max(np.abs(got - want) / want) <= 1e-10
