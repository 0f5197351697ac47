"""Trees of chains, nodes with a single child, bit for bit against the oracle: levels
whose parents are all such, levels that mix them with others in a chunk of 256
children, and a few of them, which take the ordinary fold."""
import numpy as np
import pytest

import oracle
from tests.gpu_cases import compare_tree, gpu_run, log

pytestmark = pytest.mark.gpu


def _places(rng, m, copies):
    return np.repeat(rng.uniform(-1, 1, (m, 3)), copies, axis=0)


@pytest.mark.parametrize("places,copies,others,n_crit,n_leaf", [
    (400, 20, 0, 16, 16),       # 400 chains to the deepest level; leaves beyond n_crit are groups
    (129, 2, 0, 1, 1),          # just enough of them to leave the ordinary fold
    (128, 2, 0, 4, 1),          # just too few
    (150, 18, 3000, 64, 16),    # beside a tree without duplicates
    (300, 2, 600, 4, 1),
    (257, 40, 0, 64, 16)])      # more than a chunk; the chains lie below the groups
def test_chains(places, copies, others, n_crit, n_leaf):
    from paper_1506_04553_amd import P3T
    rng = np.random.default_rng(places)
    pos = np.concatenate((_places(rng, places, copies), rng.uniform(-1, 1, (others, 3))))
    mass = rng.uniform(0.5, 2.0, len(pos))
    p = dict(eps=1e-3, r_in=0.001, r_out=0.01, theta=0.6, r_search=0.011, n_crit=n_crit,
             n_leaf=n_leaf)
    log(f"chains: {places} places of {copies}, {others} others")
    ctx = P3T(0)
    compare_tree(gpu_run(ctx, pos, mass, p), oracle.Tree(pos, mass, p))
    ctx.close()

