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
