"""The direct sums at the edges of their block sizes.

Blocks of 64 particles up to 5 000, of 256 up to 49 152, then of 1 024: sizes
around whole blocks, odd and even numbers of blocks (an even number meets the
pairs at half its distance once), a single particle over; and a call captured
into a graph, which takes the one-sided kernel.  Against the definition in FP64
(torch, every pair), with the tolerance of the same terms in another order.
"""
import pytest

from tests.gpu_cases import log

pytestmark = pytest.mark.gpu

TOL = 1e-12
R = dict(r_in=0.02, r_out=0.2)


def _cluster(n):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    pos = torch.randn(n, 3, generator=g, device="cuda", dtype=torch.float64)
    mass = torch.rand(n, generator=g, device="cuda", dtype=torch.float64) / n
    return pos, mass


def _rows(pos, mass, mode, eps, rows):
    """Sums of the given particles, and those of the plain Newton terms' sizes."""
    import torch
    d = pos[None] - pos[rows][:, None]
    s = torch.sqrt((d * d).sum(-1) + eps * eps)
    self_ = torch.zeros_like(s, dtype=torch.bool)
    self_[torch.arange(len(rows)), rows] = True
    m = torch.where(self_, 0.0, mass[None])
    g = R["r_in"] / R["r_out"]
    y = s / R["r_out"]
    x = ((y - g) / (1 - g)).clamp(0, 1)
    K = x ** 4 * (35 + x * (-84 + x * (70 - 20 * x)))
    # W/y = 1 + integral_y^1 K(t)/t^2 dt by Gauss-Legendre on [max(y, g), 1]
    import numpy as np
    gx, gw = np.polynomial.legendre.leggauss(40)
    lo = y.clamp(g, 1.0)
    wy = torch.ones_like(y)
    for a, b in zip(gx, gw):
        t = lo + (1 - lo) * 0.5 * (a + 1)
        u = (t - g) / (1 - g)
        wy += 0.5 * b * (1 - lo) * u ** 4 * (35 + u * (-84 + u * (70 - 20 * u))) / t ** 2
    W = torch.where(y >= 1, 1.0, wy * y)
    if mode == "newton":
        K, W = torch.ones_like(K), torch.ones_like(W)
    if mode == "hard":
        K, W = 1 - K, 1 - W
    f = m / s ** 3
    return ((f * K)[..., None] * d).sum(1), -(m * W / s).sum(1), (f[..., None] * d).abs().sum(1), (m / s).sum(1)


@pytest.mark.parametrize("mode", ["newton", "soft", "hard"])
@pytest.mark.parametrize("n", [1, 64, 65, 128, 193, 5000, 5001, 5120, 5121, 49152, 49153, 51201])
def test_direct_block_edges(n, mode):
    import torch
    from paper_1506_04553_amd import P3T
    pos, mass = _cluster(n)
    eps = 1e-3
    ctx = P3T(0)
    acc, pot = ctx.direct(pos, mass, mode, eps=eps, theta=0.5, r_search=0.22, **R)
    again, _ = ctx.direct(pos, mass, mode, want_pot=False, eps=eps, theta=0.5, r_search=0.22, **R)
    ctx.close()
    rows = torch.arange(n, device="cuda") if n <= 200 else torch.cat(
        [torch.arange(70), torch.arange(n // 2 - 35, n // 2 + 35), torch.arange(n - 70, n)]).cuda()
    ra, rp, sa, sp = _rows(pos, mass, mode, eps, rows)
    ea = float(((acc[rows] - ra).abs() / sa.clamp_min(1e-300)).max())
    ep = float(((pot[rows] - rp).abs() / sp.clamp_min(1e-300)).max())
    log(f"direct {mode} n={n}: acc {ea:.1e} pot {ep:.1e}")
    assert ea < TOL and ep < TOL
    assert torch.equal(acc, again)


def test_direct_captured():
    import torch
    from paper_1506_04553_amd import P3T
    pos, mass = _cluster(3000)
    kw = dict(eps=1e-3, theta=0.5, r_search=0.22, **R)
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    ctx = P3T(0, stream=stream)
    with torch.cuda.stream(stream):
        ctx.direct(pos, mass, "soft", **kw)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        acc, pot = ctx.direct(pos, mass, "soft", **kw)
    for k in range(3):
        pos.mul_(1.0 - 0.01 * k)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            ea, ep = ctx.direct(pos, mass, "soft", **kw)
        torch.cuda.synchronize()
        assert float((acc - ea).norm() / ea.norm()) < TOL
        assert float((pot - ep).norm() / ep.norm()) < TOL
    ctx.close()
