"""The lists of a tree of more than 50000 nodes, whose walk accepts most cells
without reading their boxes, bit for bit against the oracle's: opening angles
from those that let most cells be told from afar to the largest that lets any,
and one that lets none, with search radii from far below the cells' sizes to far
above, where the boxes decide."""
import numpy as np
import pytest

import oracle
from inputs import plummer
from tests.gpu_cases import compare_tree, gpu_run, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("theta,h", [(0.3, 1e-4), (0.5, 0.05), (0.5, 0.6), (0.57, 0.01),
                                     (0.9, 0.02)])
def test_lists_of_many_nodes(theta, h):
    from paper_1506_04553_amd import P3T
    c = plummer(60000, 8)
    p = dict(eps=1e-3, r_in=0.09 * h, r_out=0.9 * h, theta=theta, r_search=h, n_crit=64, n_leaf=1)
    ctx = P3T(0)
    for _ in range(2):                  # two-pass lists, then lists of fixed stride
        g = gpu_run(ctx, c.pos, c.mass, p, want_neighbors=False)
    t = oracle.Tree(c.pos, c.mass, p)
    log(f"theta {theta} h {h}: {t.n_nodes} nodes, {t.n_groups} groups")
    assert t.n_nodes > 50000
    compare_tree(g, t, groups_sample=range(0, t.n_groups, 17))
    ctx.close()


@pytest.mark.parametrize("masses", ["subnormal", "overflow", "far out"])
def test_lists_where_centres_leave_their_boxes(masses):
    """Centres of mass away from the members: masses of a few times the smallest
    number, masses whose products with the positions overflow, and positions whose
    rounding is as large as the deepest cells.  The lists of neighbours are complete
    all the same."""
    from paper_1506_04553_amd import P3T
    c = plummer(60000, 9)
    n, rng, h = len(c.mass), np.random.default_rng(10), 0.05
    pos, mass = c.pos, c.mass
    if masses == "subnormal":
        mass = rng.integers(1, 40, n) * 5e-324
    elif masses == "overflow":
        pos, mass, h = c.pos * 1e20, rng.uniform(0.5, 1.0, n) * 1e290, 0.05 * 1e20
    else:
        pos, h = c.pos + 2.0 ** 36, 2.0 ** -6
    p = dict(eps=1e-3, r_in=0.09 * h, r_out=0.9 * h, theta=0.5, r_search=h, n_crit=64, n_leaf=1)
    ctx = P3T(0)
    for _ in range(2):
        g = gpu_run(ctx, pos, mass, p, want_arrays=False)
    ctx.close()
    t = oracle.Tree(pos, mass, p)
    off, idx = t.neighbors()
    log(f"{masses}: {t.n_nodes} nodes, {len(idx)} pairs, {len(g['nbr_idx'])} found")
    assert t.n_nodes > 50000 and len(idx) > 0
    assert np.array_equal(g["nbr_off"], off) and np.array_equal(g["nbr_idx"], idx)
