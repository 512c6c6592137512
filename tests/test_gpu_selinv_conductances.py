"""Sparse-direct maps of stacks whose conductances are spread over nine decades,
drawn edge by edge: the panels are eliminated by explicit inverses, which lose
nothing on M-matrices.  G's diagonal entries alone are rounded sums of
conductances up to 1e9 apart, so no float64 factorisation of G is exact there;
the measure is a Cholesky factorisation and the same recurrences in float64
(oracle/selinv.py), both against unit solves refined with extended-precision
residuals taken edge by edge.  The two eliminate in different orders with errors
that are sums of the same kind, so either may be ahead on one stack: the bar is
ten times the Cholesky's worst error, and 1e-12 where that is smaller."""
import numpy as np
import pytest
import scipy.sparse.linalg as spla

from oracle import reff_oracle as ro
from oracle import selinv as osel
from paper_2607_05818_amd import gen

pytestmark = pytest.mark.gpu


def _refined(d, nodes):
    u, v, w = ro.edge_list_fast(d)
    w = w.astype(np.longdouble)
    G, free = ro.grounded(d, True)
    lu = spla.splu(G.tocsc(), permc_spec="MMD_AT_PLUS_A")
    grounded = np.ones(gen.n_nodes(d), bool)
    grounded[free] = False
    E = np.zeros((gen.n_nodes(d), len(nodes)), np.longdouble)
    E[nodes, np.arange(len(nodes))] = 1
    X = np.zeros_like(E)
    for _ in range(12):
        cur = (X[u] - X[v]) * w[:, None]
        res = E.copy()
        np.add.at(res, u, -cur)
        np.add.at(res, v, cur)
        step = lu.solve(res[free].astype(np.float64))
        X[free] += step
    assert np.abs(step).max() <= 1e-17 * np.abs(X).max()
    return X[nodes, np.arange(len(nodes))]


def spread_stack(nt, nx, ny, decades):
    d = gen.small_random_desc(3, nt, nx, ny, 12 if nt > 1 else 0, 5)
    rng = np.random.default_rng([nt, nx, ny])
    for k in ("gx", "gy", "tsv_g"):
        d[k] = d[k] * 10.0 ** rng.uniform(-decades / 2, decades / 2, d[k].shape)
    return d


@pytest.mark.parametrize("decades", [4, 9])
@pytest.mark.parametrize("nt,nx,ny", [(1, 40, 30), (3, 24, 24), (4, 64, 64), (2, 3, 200)])
def test_errors_stay_those_of_cholesky(nt, nx, ny, decades):
    from paper_2607_05818_amd import reff
    d = spread_stack(nt, nx, ny, decades)
    nodes = gen.sample_free_nodes(d, 60, 3)
    want = _refined(d, nodes)
    chol = float(np.max(np.abs(osel.diag_full(d)[nodes] - want) / want))
    print("[case] selinv conductances", nt, nx, ny, decades, flush=True)
    h = reff.reff_build_pdn(d)
    got, _ = reff.reff_selinv_diag(h)
    h.close()
    err = float(np.max(np.abs(got[nodes] - want) / want))
    print(f"Cholesky {chol:.2e}, here {err:.2e}", flush=True)
    assert err <= max(10 * chol, 1e-12)
