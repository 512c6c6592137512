"""The paths of the pair calls that the sizes of the other tests do not reach:
the cross term over several 64-column steps in one, two, three and four parts,
direct products with several 64-point blocks and with fewer m segments than the
allocating call uses, and the reduced system over tiers served by direct
products."""
import numpy as np
import pytest

from oracle import reff_oracle as ro
from tests.test_gpu_grid_table import _points, _want
from tests.test_gpu_reduced_pairs import _desc, _stack
from tests.test_gpu_reduced_tiles import _refined_floating_pairs

pytestmark = pytest.mark.gpu


# p = 100: K = 200, three full steps and one of 8 columns
@pytest.mark.parametrize("m,n,parts", [(1100, 1000, 1), (900, 900, 2), (700, 800, 3), (90, 70, 4)])
def test_cross_term_over_several_steps(m, n, parts):
    """Against the oracle's floating pairs of every 13th bump and load.  Both
    sides are float64 direct solves of systems whose condition stays below 1e4
    at these sizes, so the bar is 1e-10."""
    from paper_2607_05818_amd import reff
    tiles = -(-m // 64) * -(-n // 64)
    assert max(1, min(4, 512 // tiles)) == parts
    nx, ny, d, p = 60, 55, 2, 100
    rng = np.random.default_rng([m, n])
    r_t, s_t, txy, tr, _, _ = _stack(31, d, nx, ny, p, 1, 1)
    pick = lambda c: rng.permutation(nx * ny)[:c]  # noqa: E731
    b, c = pick(m), pick(n)
    bump = np.stack([b % nx, b // nx], 1).astype(np.int32)
    load = np.stack([c % nx, c // nx], 1).astype(np.int32)
    want = ro.pairs(_desc(nx, ny, r_t, s_t, txy, tr), b[::13], (d - 1) * nx * ny + c[::13], mode=ro.FLOATING)
    print("[case] cross term", m, n, parts, flush=True)
    got = reff.reff_reduced_pairs(nx, ny, r_t, s_t, txy, tr, bump, load)[::13, ::13]
    assert np.max(np.abs(got - want) / want) <= 1e-10


@pytest.mark.parametrize("d,p", [(3, 20), (2, 70), (4, 44)])
def test_tsv_resistances_over_twelve_decades_entry_by_entry(d, p):
    """Every pair by itself, not against the largest: the pairs of a stack lie
    within a factor of seven of each other and the largest error is below 6e-11
    of the largest pair, so 1e-9 holds for each."""
    from paper_2607_05818_amd import reff
    nx = 40
    rng = np.random.default_rng(d * 100 + p)
    at = rng.choice(400, p, replace=False)
    xy = np.stack([at % 20 + 3, at // 20 + 5], 1).astype(np.int32)
    tr = 10.0 ** rng.uniform(-6, 6, (p, d - 1))
    r_t, s_t = np.linspace(0.5, 2, d), np.linspace(1, 3, d)
    bump = rng.integers(0, nx, (9, 2)).astype(np.int32)
    load = rng.integers(0, nx, (17, 2)).astype(np.int32)
    ids = lambda a, t: t * nx * nx + a[:, 1].astype(np.int64) * nx + a[:, 0]  # noqa: E731
    want = _refined_floating_pairs(_desc(nx, nx, r_t, s_t, xy, tr),
                                   np.concatenate([ids(bump, 0), ids(load, d - 1)]), 9)
    print("[case] reduced twelve decades", d, p, flush=True)
    got = reff.reff_reduced_pairs(nx, nx, r_t, s_t, xy, tr, bump, load)
    assert np.max(np.abs(got - want) / want) <= 1e-9


def test_direct_products_of_several_blocks():
    """70 points of a 20000 x 3 tier, two blocks of 64, by direct products in
    both entry points; the bar is that of the other Eq. 3 tests."""
    from paper_2607_05818_amd import reff
    rng = np.random.default_rng(70)
    xy = _points(rng, 20000, 3, 70)
    want = _want(20000, 3, 0.7, 1.9, xy)
    off = ~np.eye(len(xy), dtype=bool)
    print("[case] direct products, 70 points", flush=True)
    for fn in (reff.reff_grid_pairs, reff.reff_grid_pairs_noalloc):
        got = fn(20000, 3, 0.7, 1.9, xy)
        assert np.array_equal(got, got.T)
        assert np.max(np.abs(got[off] - want[off]) / want[off]) <= 1e-11


def test_direct_products_where_the_table_does_not_fit():
    """2100 x 2100 with 100 points: the table and its inputs are more than the
    64 MiB of the call without allocation, whose direct products then run in
    fewer m segments than they would have; the allocating call takes the table.
    The first four points against extended precision, all pairs against each
    other."""
    from paper_2607_05818_amd import reff
    M, P = 2100, 100
    r256 = lambda b: -(-b // 256) * 256  # noqa: E731
    table = (2 * r256(16 * M) + r256(8 * (M + 1) * (M - 1)) + r256(8 * (M + 1) ** 2) + r256(16 + 8 * P) +
             r256(8 * P * P))
    fixed = r256(8 * P) + r256(8 * (M - 1) ** 2) + r256(8 * P * (M - 1)) + r256(8 * P * P)
    segments = -(-2048 // 3)  # 3 block pairs
    assert table > 64 << 20 and fixed + 8 * P * P <= 64 << 20 < fixed + segments * 8 * P * P
    rng = np.random.default_rng(5)
    xy = _points(rng, M, M, P)
    want = _want(M, M, 0.7, 1.9, xy[:4])
    print("[case] grid paths 2100", flush=True)
    a = reff.reff_grid_pairs(M, M, 0.7, 1.9, xy)
    b = reff.reff_grid_pairs_noalloc(M, M, 0.7, 1.9, xy)
    off = ~np.eye(P, dtype=bool)
    assert np.max(np.abs(a[off] - b[off]) / a[off]) <= 1e-11
    off = off[:4, :4]
    for got in (a, b):
        assert np.max(np.abs(got[:4, :4][off] - want[off]) / want[off]) <= 1e-11


def test_reduced_system_over_direct_products():
    """Tiers of 14000 x 3 with 76 endpoints, for which direct products are
    cheaper than the table.  Eq. 3 is good to 1e-11 of the intra-die resistances,
    9e3 ohm at most, and the smallest pair is 48 ohm: 2e-9, and the bar 1e-8."""
    from paper_2607_05818_amd import reff
    nx, d, p = 14000, 3, 70
    r_t, s_t, txy, tr, bump, load = _stack(77, d, nx, 3, p, 5, 6)
    ids = lambda a, t: t * nx * 3 + a[:, 1].astype(np.int64) * nx + a[:, 0]  # noqa: E731
    want = _refined_floating_pairs(_desc(nx, 3, r_t, s_t, txy, tr),
                                   np.concatenate([ids(bump, 0), ids(load, d - 1)]), 5)
    print("[case] reduced over direct products", flush=True)
    got = reff.reff_reduced_pairs(nx, 3, r_t, s_t, txy, tr, bump, load)
    assert np.max(np.abs(got - want) / want) <= 1e-8
