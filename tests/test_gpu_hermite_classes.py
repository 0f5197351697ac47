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


def _components(rng, sizes, cliques, stars=0, isolated=0):
    """Members of each component around its own centre, shuffled over the arrays;
    every member lists the two beside it, or (the first `cliques`) all others, or
    (the first `stars`) the two beside it and the first one, which lists all.
    `isolated` particles more list nothing."""
    n = int(sum(sizes)) + isolated
    slot = rng.permutation(n)
    pos, rows, b = rng.uniform(-9, -1, (n, 3)), [np.zeros(0, np.int64)] * n, 0
    for c, m in enumerate(sizes):
        me = slot[b:b + m]
        d = rng.uniform(-1e-3, 1e-3, (m, 3))
        d[:, 0] += 0.006 * np.arange(m) if c >= cliques else 0.0
        pos[me] = np.array([(c % 32) * 1.0, (c // 32) * 1.0, 0.0]) + d
        for k in range(m):
            nb = np.arange(m) if c < cliques else np.arange(max(k - 1, 0), min(k + 2, m))
            if c < stars:
                nb = np.unique(np.append(nb, 0)) if k else np.arange(m)
            rows[me[k]] = np.sort(me[nb[nb != k]])
        b += m
    off = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
    return pos, off, np.concatenate(rows).astype(np.int32)


@pytest.mark.parametrize("sizes,cliques,n", [
    ([63, 31, 32, 63, 64, 8, 1 + 6], 1, 0),
    ([63, 32, 64] + [32] * 511 + [63, 31, 31, 16, 15], 2, 0),   # 515 of 32 and more
    # the search for components in one workgroup: its last n and the first beyond,
    # and more list entries than it takes (370 x 369)
    ([2] * 4000 + [7, 33, 3], 0, 16384),
    ([2] * 4000 + [7, 33, 3], 0, 16385),
    ([370, 2, 5], 1, 0),
    ([2], 0, 2),
])
def test_size_classes_match_oracle(ctx, sizes, cliques, n):
    import torch
    rng = np.random.default_rng(5)
    pos, off, idx = _components(rng, sizes, cliques, isolated=max(n - sum(sizes), 0))
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


@pytest.mark.parametrize("special,isolated", [(0, 0), (3, 0), (0, 13000)])
def test_giant_components_match_oracle(ctx, special, isolated):
    """Components that advance by grid-wide launches, at the edges of their class
    (1024 members, and 1023 beside them), with the members of three of them in one
    run of 64, with rows longer than a workgroup takes at a time, with a component
    that needs far fewer block steps than the other, with special particles, and
    beside so many isolated ones that the components are found by many launches."""
    import torch
    rng = np.random.default_rng(6)
    pos, off, idx = _components(rng, [1101, 1024, 1025, 1023, 2, 40], 0, stars=1,
                                isolated=isolated)
    n = len(pos)
    vel = rng.normal(scale=0.02, size=(n, 3))
    mass = rng.uniform(0.5e-6, 1.5e-6, n)
    p = dict(eps=1e-4, r_in=0.001, r_out=0.01, theta=0.5, r_search=0.011, n_crit=64, n_leaf=16)
    hk = dict(dt_soft=2.0 ** -7, dt_max=2.0 ** -9, eta=0.01, eta_s=0.001, a0=1e-5,
              max_block_steps=200000)
    kinds = dict(n_special=special, r_in_ns=0.004, r_out_ns=0.02, r_search_ns=0.03, eps_ns=1e-3,
                 split_ss=0, r_in_ss=0.0, r_out_ss=1.0, r_search_ss=1.0, eps_ss=0.0,
                 eta_sp=0.003, eta_s_sp=0.0003) if special else None
    okinds = {k: w for k, w in kinds.items() if "search" not in k} if special else None
    args = [torch.from_numpy(a).cuda() for a in (mass, off, idx)]
    x, v = torch.from_numpy(pos.copy()).cuda(), torch.from_numpy(vel.copy()).cuda()
    ns, st = ctx.hermite_hard(x, v, *args, hk, kinds=kinds, **p)
    okw = {k: hk[k] for k in ("dt_soft", "dt_max", "eta", "eta_s", "a0")}
    ox, ov, ons, _ = oracle.hermite(pos, vel, mass, off, idx, p["eps"], p["r_in"], p["r_out"],
                                    kinds=okinds, **okw)
    log(f"giants, {special} special: {st}")
    assert st["max_cluster"] == 1101 and st["max_block_steps"] > 32
    assert np.array_equal(ns.cpu().numpy(), ons)
    assert np.array_equal(x.cpu().numpy(), ox) and np.array_equal(v.cpu().numpy(), ov)
    # a bound below the steps of the longest component ends the call
    from paper_1506_04553_amd.p3t import P3TError
    with pytest.raises(P3TError):
        ctx.hermite_hard(torch.from_numpy(pos.copy()).cuda(), torch.from_numpy(vel.copy()).cuda(),
                         *args, {**hk, "max_block_steps": 1}, kinds=kinds, **p)
