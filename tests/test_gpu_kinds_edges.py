"""Neighbour lists and soft pulls with special particles where the launches and
the prefix sums change shape: one particle to a whole workgroup and one more,
the largest count that a single workgroup scans and the first beyond, no normal
particle, and lists of more than one workgroup's chunk of hits.  The lists are
whole numbers and must be the definition's; the sums are FP64 in another order."""
import numpy as np
import pytest

from oracle import direct
from tests.gpu_cases import log, rel_rms

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1506_04553_amd import P3T
    c = P3T(0)
    yield c
    c.close()


@pytest.mark.parametrize("n,n_special,r", [
    (1, 1, 0.5), (2, 1, 2.0), (3, 3, 0.9), (1024, 1, 0.6), (1025, 2, 0.6), (1026, 1, 3.0),
    (16383, 2, 0.4), (16384, 3, 0.4), (2500, 2, 3.0)])
def test_kinds_lists_and_pulls(ctx, n, n_special, r):
    import torch
    rng = np.random.default_rng(n)
    pos = rng.uniform(-1, 1, (n, 3))
    mass = rng.uniform(0.5, 1.5, n) / n
    kinds = dict(n_special=n_special, r_in_ns=0.05, r_out_ns=0.3, r_search_ns=r, eps_ns=1e-3,
                 split_ss=1, r_in_ss=0.1, r_out_ss=0.5, r_search_ss=0.8, eps_ss=1e-3,
                 eta_sp=0.03, eta_s_sp=0.003)
    p = dict(eps=1e-3, r_in=0.01, r_out=0.1, theta=0.5, r_search=0.11, n_crit=64, n_leaf=16)
    dpos, dmass = torch.from_numpy(pos).cuda(), torch.from_numpy(mass).cuda()
    # the normal particles' own lists: a ring
    m = n - n_special
    nn = [np.unique([(i - 1) % m, (i + 1) % m]) if m > 2 else np.zeros(0, int) for i in range(m)]
    nn_off = np.concatenate([[0], np.cumsum([len(x) for x in nn])]).astype(np.int64)
    nn_idx = np.concatenate(nn + [np.zeros(0, int)]).astype(np.int32)
    if len(nn_idx) == 0:
        nn_idx = np.zeros(1, np.int32)
    off, idx = ctx.kinds_neighbors(dpos, kinds, torch.from_numpy(nn_off).cuda(),
                                   torch.from_numpy(nn_idx).cuda())
    d2 = lambda b: ((pos[b] - pos)[:, 0] ** 2 + (pos[b] - pos)[:, 1] ** 2) + (pos[b] - pos)[:, 2] ** 2
    near = {b: d2(b) < r * r for b in range(m, n)}
    rows = [np.concatenate([nn[i], [b for b in range(m, n) if near[b][i]]]).astype(int)
            for i in range(m)]
    for b in range(m, n):
        hit = near[b].copy()
        hit[m:] = d2(b)[m:] < 0.8 * 0.8
        hit[b] = False
        rows.append(np.flatnonzero(hit))
    ref = np.concatenate([[0], np.cumsum([len(x) for x in rows])])
    log(f"kinds n={n}: {ref[-1]} entries, special rows {[len(x) for x in rows[m:]]}")
    assert np.array_equal(off.cpu().numpy(), ref)
    assert np.array_equal(idx.cpu().numpy()[:ref[-1]], np.concatenate(rows))
    acc = torch.zeros((n, 3), dtype=torch.float64, device="cuda")
    pot = torch.zeros(n, dtype=torch.float64, device="cuda")
    ctx.kinds_soft(dpos, dmass, acc, pot, kinds, **p)
    oa, op = direct.kinds_soft(pos, mass, p["eps"], p["r_in"], p["r_out"], kinds)
    if n > 1:   # sums of at most n terms of one sign scale: n eps is below 4e-12
        assert rel_rms(acc.cpu().numpy(), oa) < 4e-12 and rel_rms(pot.cpu().numpy(), op) < 4e-12
