"""The size classes of the block-timestep integration at their edges: components
of 31, 32, 63 and 64 members, with few of 32 to 255 (those of 32 to 63 members
take a workgroup each) and with more than run at once (they take a wavefront
each), with short lists and with lists that outgrow their LDS area.  Positions,
velocities and step counts must be the oracle's bit for bit: the classes differ
in which lanes evaluate a term, not in the order in which terms are added."""
import numpy as np
import pytest

import oracle
from tests.gpu_cases import log

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1506_04553_amd import P3T
    c = P3T(0)
    yield c
    c.close()


def _components(rng, sizes, cliques):
    """Members of each component around its own centre, shuffled over the arrays;
    every member lists the two beside it, or (the first `cliques`) all others."""
    n = int(sum(sizes))
    slot = rng.permutation(n)
    pos, rows, b = np.empty((n, 3)), [None] * n, 0
    for c, m in enumerate(sizes):
        me = slot[b:b + m]
        d = rng.uniform(-1e-3, 1e-3, (m, 3))
        d[:, 0] += 0.006 * np.arange(m) if c >= cliques else 0.0
        pos[me] = np.array([(c % 32) * 1.0, (c // 32) * 1.0, 0.0]) + d
        for k in range(m):
            nb = np.arange(m) if c < cliques else np.arange(max(k - 1, 0), min(k + 2, m))
            rows[me[k]] = np.sort(me[nb[nb != k]])
        b += m
    off = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
    return pos, off, np.concatenate(rows).astype(np.int32)


@pytest.mark.parametrize("sizes,cliques", [
    ([63, 31, 32, 63, 64, 8, 1 + 6], 1),
    ([63, 32, 64] + [32] * 511 + [63, 31, 31, 16, 15], 2),   # 515 of 32 and more
])
def test_size_classes_match_oracle(ctx, sizes, cliques):
    import torch
    rng = np.random.default_rng(5)
    pos, off, idx = _components(rng, sizes, cliques)
    n = len(pos)
    vel = rng.normal(scale=0.02, size=(n, 3))
    mass = rng.uniform(0.5e-6, 1.5e-6, n)
    p = dict(eps=1e-4, r_in=0.001, r_out=0.01, theta=0.5, r_search=0.011, n_crit=64, n_leaf=16)
    hk = dict(dt_soft=2.0 ** -7, dt_max=2.0 ** -9, eta=0.1, eta_s=0.01, a0=1e-5,
              max_block_steps=200000)
    x, v = torch.from_numpy(pos.copy()).cuda(), torch.from_numpy(vel.copy()).cuda()
    ns, st = ctx.hermite_hard(x, v, torch.from_numpy(mass).cuda(), torch.from_numpy(off).cuda(),
                              torch.from_numpy(idx).cuda(), hk, **p)
    ox, ov, ons, _ = oracle.hermite(pos, vel, mass, off, idx, p["eps"], p["r_in"], p["r_out"],
                                    **{k: hk[k] for k in ("dt_soft", "dt_max", "eta", "eta_s",
                                                          "a0")})
    log(f"{len(sizes)} components: {st}")
    assert st["n_clusters"] == len(sizes) and st["max_cluster"] == max(sizes)
    assert np.array_equal(ns.cpu().numpy(), ons)
    assert np.array_equal(x.cpu().numpy(), ox) and np.array_equal(v.cpu().numpy(), ov)
