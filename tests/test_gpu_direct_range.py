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
