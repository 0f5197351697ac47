"""The whole tree, bit for bit against the oracle, at the edges of the kernels that
build it: particle counts around a tile of the group records (4096), children
around a chunk of the moments (256, with parents across the boundary), full
octants, and leaves as groups."""
import numpy as np
import pytest

import oracle
from inputs import plummer
from tests.gpu_cases import compare_tree, gpu_run, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n,n_crit,n_leaf", [
    ("plummer", 4095, 64, 16), ("plummer", 4096, 16, 16), ("plummer", 4097, 1, 1),
    ("plummer", 8193, 64, 1), ("plummer", 30000, 40, 3), ("grid", 512, 8, 8),
    ("grid", 4096, 1, 1)])
def test_tree_at_edges(kind, n, n_crit, n_leaf):
    from paper_1506_04553_amd import P3T
    if kind == "grid":      # full octants: eight children each
        m = round(n ** (1 / 3))
        pos = np.stack(np.meshgrid(*[np.arange(m)] * 3, indexing="ij"), -1).reshape(-1, 3) / m
    else:
        pos = plummer(n, 71).pos
    pos = np.ascontiguousarray(pos, dtype=np.float64)
    mass = np.random.default_rng(72).uniform(0.5, 2.0, n)
    p = dict(eps=1e-3, r_in=0.001, r_out=0.01, theta=0.6, r_search=0.011, n_crit=n_crit,
             n_leaf=n_leaf)
    log(f"tree edges {kind} n={n} n_crit={n_crit} n_leaf={n_leaf}")
    ctx = P3T(0)
    compare_tree(gpu_run(ctx, pos, mass, p), oracle.Tree(pos, mass, p))
    ctx.close()
