"""Builds of one context whose particles suit the sort by leading bits and whose do
not, each of another number: Morton order bit for bit against the oracle."""
import numpy as np
import pytest

import oracle
from tests.gpu_cases import log
from tests.test_gpu_sort_long import P, _runs

pytestmark = pytest.mark.gpu


def test_sorts_in_turn():
    import torch
    from paper_1506_04553_amd import P3T
    ctx = P3T(0)
    rng = np.random.default_rng(12)
    for k in range(24):
        n = 24000 + 211 * k           # the first ones are ranked
        pos = _runs(n, [n // 2] if k in (0, 4, 5, 23) else [64, 40], rng)
        mass = np.full(n, 1.0 / n)
        ctx.build_tree(torch.from_numpy(pos).cuda(), torch.from_numpy(mass).cuda(), **P)
        key, perm = oracle.Tree(pos, mass, P).keys()
        log(f"build {k} of {n}")
        np.testing.assert_array_equal(ctx.copy_array("perm").astype(np.int64), perm)
        np.testing.assert_array_equal(ctx.copy_array("sorted_keys"), key[perm])
    ctx.close()
