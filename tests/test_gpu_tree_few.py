"""The whole tree, bit for bit against the oracle, at the particle counts where the
build's launches change: up to 12288 particles the topology adds up its blocks'
node counts itself, and the host the levels'."""
import numpy as np
import pytest

import oracle
from inputs import plummer
from tests.gpu_cases import compare_tree, gpu_run, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,n_crit,n_leaf", [
    (1, 8, 8), (17, 16, 16), (257, 4, 1), (4095, 64, 16), (4096, 2, 1), (8191, 64, 16),
    (8192, 64, 16), (12288, 32, 4), (12289, 32, 4)])
def test_tree_at_launch_changes(n, n_crit, n_leaf):
    from paper_1506_04553_amd import P3T
    pos = np.ascontiguousarray(plummer(max(n, 2), 73).pos[:n], dtype=np.float64)
    mass = np.random.default_rng(74).uniform(0.5, 2.0, n)
    p = dict(eps=1e-3, r_in=0.001, r_out=0.01, theta=0.6, r_search=0.011, n_crit=n_crit,
             n_leaf=n_leaf)
    log(f"n={n} n_crit={n_crit} n_leaf={n_leaf}")
    ctx = P3T(0)
    t = oracle.Tree(pos, mass, p)
    for _ in range(2):
        compare_tree(gpu_run(ctx, pos, mass, p, want_neighbors=False), t)
    ctx.close()
