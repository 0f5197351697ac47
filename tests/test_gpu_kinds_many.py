"""Soft pulls with many special particles, where several threads take a normal
particle's sum: the numbers of special ones at which that changes, and as many as do
not divide among the threads; and that the launch does not wait for those sums."""
import numpy as np
import pytest

from oracle import direct
from tests.gpu_cases import log, rel_rms

pytestmark = pytest.mark.gpu
P = dict(eps=1e-3, r_in=0.01, r_out=0.1, theta=0.5, r_search=0.11, n_crit=64, n_leaf=16)


def _kinds(n_special):
    return dict(n_special=n_special, r_in_ns=0.05, r_out_ns=0.3, r_search_ns=0.3, eps_ns=1e-3,
                split_ss=1, r_in_ss=0.1, r_out_ss=0.5, r_search_ss=0.8, eps_ss=1e-3,
                eta_sp=0.03, eta_s_sp=0.003)


@pytest.mark.parametrize("n,n_special", [(1025, 1), (1026, 2), (1032, 8), (1033, 9), (100, 93),
                                         (3000, 2), (3000, 3), (3000, 24), (3000, 25), (3000, 77),
                                         (64, 64)])
def test_pulls_of_many(n, n_special):
    import torch
    from paper_1506_04553_amd import P3T
    rng = np.random.default_rng(n + n_special)
    pos, mass = rng.uniform(-1, 1, (n, 3)), rng.uniform(0.5, 1.5, n) / n
    base, kinds = rng.normal(size=(n, 3)), _kinds(n_special)
    ctx = P3T(0)
    acc = torch.from_numpy(base.copy()).cuda()
    pot = torch.zeros(n, dtype=torch.float64, device="cuda")
    ctx.kinds_soft(torch.from_numpy(pos).cuda(), torch.from_numpy(mass).cuda(), acc, pot, kinds, **P)
    ctx.close()
    oa, op = direct.kinds_soft(pos, mass, P["eps"], P["r_in"], P["r_out"], kinds)
    oa[:n - n_special] += base[:n - n_special]
    ea, ep = rel_rms(acc.cpu().numpy(), oa), rel_rms(pot.cpu().numpy(), op)
    log(f"kinds n={n}, {n_special} special: acc {ea:.1e} pot {ep:.1e}")
    assert ea < 4e-12 and ep < 4e-12     # sums of at most n terms of one sign scale


def test_many_pulls_side_by_side():
    """300 special particles of 6000 take less than four times as long as 16 (twice as
    long here, 14 times with one thread to each normal particle)."""
    import torch
    from paper_1506_04553_amd import P3T
    n, rng = 6000, np.random.default_rng(1)
    pos, mass = torch.from_numpy(rng.normal(size=(n, 3))).cuda(), torch.ones(n, dtype=torch.float64).cuda()
    acc, pot = torch.zeros(n, 3, dtype=torch.float64).cuda(), torch.zeros(n, dtype=torch.float64).cuda()
    ctx, took = P3T(0), {}
    for n_special in (16, 300):
        ms = []
        for _ in range(20):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(10):
                ctx.kinds_soft(pos, mass, acc, pot, _kinds(n_special), **P)
            b.record()
            b.synchronize()
            ms.append(a.elapsed_time(b))
        took[n_special] = min(ms)
    ctx.close()
    log(f"ten calls: {took}")
    assert took[300] < 4 * took[16]
