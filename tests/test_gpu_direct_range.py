"""The direct sums with masses and positions that are not finite, or of any size:
what a pair does not add stays out of both sums."""
import pytest

from tests.gpu_cases import log
from tests.test_gpu_direct_pairs import R, TOL, _cluster, _rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [200, 3000, 6000, 60000])
def test_hard_sum_beyond_cutoff(n):
    """Beyond r_out the hard part adds nothing, whatever the mass or the position."""
    import torch
    from paper_1506_04553_amd import P3T
    pos, mass = _cluster(n)
    bad = torch.tensor([0, n // 3, n // 2, n - 1]).cuda()
    good = torch.ones(n, dtype=torch.bool, device="cuda")
    good[bad] = False
    inf, nan = float("inf"), float("nan")
    pos[bad] = torch.tensor([[50.0, 0, 0], [0, 50.0, 0], [inf, 0, 0], [0, 0, 1e200]],
                            dtype=torch.float64).cuda()
    mass[bad] = torch.tensor([nan, inf, 1.0, 1.0], dtype=torch.float64).cuda()
    ctx = P3T(0)
    acc, pot = ctx.direct(pos, mass, "hard", eps=1e-3, theta=0.5, r_search=0.22, **R)
    ctx.close()
    rows = torch.arange(0, int(good.sum()), max(1, n // 200), device="cuda")
    ra, rp, sa, sp = _rows(pos[good], mass[good], "hard", 1e-3, rows)
    at = torch.nonzero(good)[rows, 0]
    ea = float(((acc[at] - ra).abs() / sa.clamp_min(1e-300)).max())
    ep = float(((pot[at] - rp).abs() / sp.clamp_min(1e-300)).max())
    log(f"hard n={n}: acc {ea:.1e} pot {ep:.1e}, {int((~torch.isfinite(acc)).sum())} not finite")
    assert bool(torch.isfinite(acc).all()) and bool(torch.isfinite(pot).all())
    assert ea < TOL and ep < TOL and bool((acc[bad] == 0).all()) and bool((pot[bad] == 0).all())


@pytest.mark.parametrize("n", [1, 2, 130, 6001, 50001])
def test_sums_of_any_size(n):
    """Clusters whose coordinates lie far out, on round numbers, without softening:
    no part of a block that holds no particle takes part."""
    import torch
    from paper_1506_04553_amd import P3T
    pos, mass = _cluster(n)
    out = []
    for scale, shift in ((1.0, 0.0), (1e18, 1e18), (1.0, 1e200)):
        x = pos * scale
        x[0] = 0.0
        x[-1] = scale * (n > 1)
        if shift < 1e100:
            x += shift
        else:                   # where only the other coordinates tell them apart
            x[:, 0] = shift
        sums = {}
        ctx = P3T(0)
        for mode in ("newton", "soft", "hard"):
            sums[mode] = ctx.direct(x, mass, mode, eps=0.0, theta=0.5, r_search=0.22 * scale,
                                    r_in=R["r_in"] * scale, r_out=R["r_out"] * scale)
        ctx.close()
        rows = torch.arange(0, n, max(1, n // 200), device="cuda")
        d = x[None] - x[rows][:, None]
        s = torch.sqrt((d * d).sum(-1))
        s[torch.arange(len(rows)), rows] = float("inf")
        f = (mass / s ** 3)[..., None] * d
        for k, (ref, size) in enumerate(((f.sum(1), f.abs().sum(1)),
                                         (-(mass / s).sum(1), (mass / s).sum(1)))):
            split = sums["soft"][k][rows] + sums["hard"][k][rows]
            for got in (sums["newton"][k][rows], split):
                err = float(((got - ref).abs() / size.clamp_min(1e-300)).max())
                out.append(err)
    log(f"n={n}: {max(out):.1e}")
    assert len(out) == 12 and all(e < TOL for e in out)
