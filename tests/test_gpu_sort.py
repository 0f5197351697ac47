"""Morton order of the particles, bit for bit against the oracle, at the edges of
the two sorts (one launch up to 8192 particles, radix passes beyond): sizes
around a wavefront and a block, many equal keys (coincident particles keep
their index order), all particles in one point, on a line, and one far away."""
import numpy as np
import pytest

import oracle
from inputs import plummer
from tests.gpu_cases import log

pytestmark = pytest.mark.gpu


def _points(kind, n):
    rng = np.random.default_rng(61)
    pos = plummer(max(n, 2), 60).pos[:n].copy()
    if kind == "repeated":
        pos = pos[rng.integers(0, max(1, n // 5), n)]
    elif kind == "point":
        pos[:] = pos[0]
    elif kind == "line":
        pos[:, 1:] = 0.25
    elif kind == "outlier":
        pos[n // 2] = 1e5
    return np.ascontiguousarray(pos)


@pytest.mark.parametrize("kind", ["plummer", "repeated", "point", "line", "outlier"])
@pytest.mark.parametrize("n", [1, 2, 63, 65, 1024, 1025, 4097, 8192, 8193, 20001])
def test_sorted_order(kind, n):
    import torch
    from paper_1506_04553_amd import P3T
    pos = _points(kind, n)
    mass = np.full(n, 1.0 / n)
    p = dict(eps=1e-3, r_in=0.001, r_out=0.01, theta=0.5, r_search=0.011, n_crit=64, n_leaf=16)
    ctx = P3T(0)
    ctx.build_tree(torch.from_numpy(pos).cuda(), torch.from_numpy(mass).cuda(), **p)
    log(f"sort {kind} n={n}")
    key, perm = oracle.Tree(pos, mass, p).keys()
    np.testing.assert_array_equal(ctx.copy_array("perm").astype(np.int64), perm)
    np.testing.assert_array_equal(ctx.copy_array("sorted_keys"), key[perm])
    ctx.close()
