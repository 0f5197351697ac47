"""Morton order bit for bit against the oracle where the keys are ordered by their
leading bits first and runs of equal leading bits then by the rest: sizes at the
first of that sort and at the edges of its last step's blocks, runs of every
length up to the longest it orders and one more (which takes the passes over all
bits), across block edges, with equal keys, and a build after such a one."""
import numpy as np
import pytest

import oracle
from tests.gpu_cases import log

pytestmark = pytest.mark.gpu
P = dict(eps=1e-3, r_in=0.001, r_out=0.01, theta=0.5, r_search=0.011, n_crit=64, n_leaf=16)


def _runs(n, lengths, rng):
    """n particles in the cube [0, 1): lower halves of cells of 2^-13 (40 bits of the
    key) with `lengths` particles each, some of them coincident, in random input
    order, the rest anywhere."""
    pos = rng.uniform(0, 1, (n, 3))
    pos[0], pos[1] = 0.0, 1.0 - 2.0 ** -20
    k = 2
    for m in lengths:
        cell = rng.integers(0, 2 ** 13, 3) / 2.0 ** 13
        pos[k:k + m] = cell + rng.uniform(0, 1, (m, 3)) * [2.0 ** -14, 2.0 ** -13, 2.0 ** -13]
        pos[k:k + m // 3] = pos[k]
        k += m
    assert k <= n
    return pos[rng.permutation(n)]


@pytest.mark.parametrize("n,lengths,whole", [
    (24577, [], False), (25600, [2, 3, 5, 64] * 40, False), (25601, [64] * 300, False),
    (25855, [65], True), (40000, list(range(2, 65)) * 4, False), (30000, [64] * 100 + [300], True),
    (33000, [33000 - 2], True)])
def test_sort_by_leading_bits(n, lengths, whole):
    import torch
    from paper_1506_04553_amd import P3T
    rng = np.random.default_rng(n)
    ctx = P3T(0)
    mass = np.full(n, 1.0 / n)
    for again in range(2):       # the second build of a context knows what the first met
        pos = _runs(n, lengths, rng)
        ctx.build_tree(torch.from_numpy(pos).cuda(), torch.from_numpy(mass).cuda(), **P)
        key, perm = oracle.Tree(pos, mass, P).keys()
        same = np.diff(np.flatnonzero(np.diff(np.concatenate([[-1], (key[perm] >> 23).astype(np.int64), [-1]]))))
        log(f"sort n={n} build {again}: longest run of the leading 40 bits {same.max()}")
        assert (same.max() > 64) == whole
        np.testing.assert_array_equal(ctx.copy_array("perm").astype(np.int64), perm)
        np.testing.assert_array_equal(ctx.copy_array("sorted_keys"), key[perm])
    ctx.close()
