"""The number of strips of a launch group: the heights of strips.h on the host
(tests/cpp/strips_check.cpp), and on the GPU tiers so narrow that their strips
are taller than 64 rows, against the oracle.  rel_tol 1e-10 (float64) and 1e-5
(mixed) are estimates, not bounds: the bars are ten times that, as in the other
parity tests."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from oracle import reff_oracle as ro
from paper_2607_05818_amd import gen

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_heights_keep_the_cap(tmp_path):
    exe = str(tmp_path / "strips_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-o", exe, os.path.join(HERE, "cpp", "strips_check.cpp")],
                   check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    print(r.stdout)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "all ok" in r.stdout


def _tier(seed, nx, ny):
    """One tier, a pad in about every 40th row."""
    rng = np.random.default_rng([seed, nx, ny])
    pads = np.stack([rng.integers(0, nx, ny // 40), rng.permutation(ny)[:ny // 40]], 1)
    return gen.make_desc(1, nx, ny, rng.uniform(0.5, 2, ny * (nx - 1)), rng.uniform(0.5, 2, (ny - 1) * nx),
                         np.zeros((0, 2), dtype=np.int32), np.zeros((0, 0)), pads)


@pytest.mark.gpu
def test_one_column():
    """17,187 strips of 64 rows; 2048 at most are allowed."""
    from paper_2607_05818_amd import reff
    d = _tier(1, 1, 1100000)
    nodes = gen.sample_free_nodes(d, 20, 3)
    print("[case] narrow tier", flush=True)
    want = ro.diag(d, nodes=nodes)
    h = reff.reff_build_pdn(d)
    got, _ = reff.reff_solve_diag(h, nodes, precision=reff.REFF_PREC_FP64, rel_tol=1e-10)
    assert np.max(np.abs(got - want) / want) <= 1e-9
    got, _ = reff.reff_solve_diag(h, nodes, precision=reff.REFF_PREC_MIXED)
    assert np.max(np.abs(got - want) / want) <= 1e-4
    h.close()


@pytest.mark.gpu
def test_group_of_narrow_plans():
    """200 plans of 33 x 3000 nodes, a full strip and one column beside it:
    18,400 strips of 64 rows in one group; 16,384 at most are allowed."""
    from paper_2607_05818_amd import reff
    two = [_tier(2, 33, 3000), _tier(3, 33, 3000)]
    nodes = [gen.sample_free_nodes(d, 8, 5 + i) for i, d in enumerate(two)]
    print("[case] narrow plans", flush=True)
    want = [ro.diag(d, nodes=v) for d, v in zip(two, nodes)]
    outs, _ = reff.reff_batch_plans([two[i % 2] for i in range(200)], [nodes[i % 2] for i in range(200)],
                                    precision=reff.REFF_PREC_MIXED)
    for i, got in enumerate(outs):
        assert np.max(np.abs(got - want[i % 2]) / want[i % 2]) <= 1e-4
