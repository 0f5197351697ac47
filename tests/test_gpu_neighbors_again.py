"""Neighbour searches one after the other, with no build and no synchronisation between
them: a search runs on a stream of its own and writes the row lengths and slots that the
call before it may still be packing from, on the context's stream."""
import numpy as np
import pytest
from scipy.spatial import cKDTree

from tests.gpu_cases import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [300, 50000])       # lengths summed by one workgroup, by two launches
@pytest.mark.parametrize("force", [False, True])  # packing behind the interaction kernel
def test_searches_back_to_back(n, force):
    import torch
    from paper_1506_04553_amd import P3T
    rng = np.random.default_rng(n)
    pos, h = rng.normal(0, 0.5, (n, 3)), 0.05 * (50000 / n) ** (1 / 3)
    p = dict(eps=4.0 / n, r_in=0.01 * h, r_out=0.1 * h, theta=0.5, r_search=h, n_crit=64, n_leaf=16)
    rows = cKDTree(pos).query_ball_point(pos, h * (1 - 1e-12))
    length = np.array([len(r) - 1 for r in rows])
    tp = torch.from_numpy(pos).cuda()
    tm = torch.full((n,), 1.0 / n, dtype=torch.float64, device="cuda")
    ctx = P3T(0)
    ctx.build_tree(tp, tm, **p)
    cap = int(ctx.neighbors()[1].numel())
    log(f"n={n}: {cap} neighbours, longest row {length.max()}")
    assert cap == length.sum() and length.max() > 8
    got = []
    for _ in range(12):
        if force:
            ctx.long_force()
        got.append(ctx.neighbors(cap))
    torch.cuda.synchronize()
    idx = np.concatenate([sorted(set(r) - {i}) for i, r in enumerate(rows)])
    for off, ix in got:
        assert np.array_equal(np.diff(off.cpu().numpy()), length)
        assert np.array_equal(ix.cpu().numpy(), idx)
    ctx.close()
