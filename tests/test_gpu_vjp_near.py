"""VJP where near particles (K, W < 1, the members themselves among them) make
up most of the particle lists.

Sizes around the 64 entries of a wavefront and the runs of 16 and 32 members,
groups of more than the 256 members staged at once, one group of everything (all
entries near, each member once its own), an inner radius beyond most pairs, and
a particle on its own.  Against the oracle's VJP on the same lists with the
tolerances of the general comparison (the same terms in another order).
"""
import numpy as np
import pytest

import oracle
from inputs import plummer
from tests.gpu_cases import log
from tests.test_gpu_vjp import _check_vjp, _gpu_vjp, ctx  # noqa: F401  (the context fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n,n_crit,r_out,with_c", [
    (15, 16, 0.5, True), (16, 16, 0.5, True), (17, 32, 0.5, False), (33, 64, 0.5, True),
    (64, 64, 0.5, True), (65, 65, 2.0, True), (257, 300, 0.5, True), (600, 600, 0.5, False),
    (1500, 128, 0.4, True), (2000, 700, 5.0, True)])
def test_vjp_near_lists(ctx, n, n_crit, r_out, with_c, precision):  # noqa: F811
    c = plummer(n, 61)
    rng = np.random.default_rng(62)
    mass = rng.uniform(0.5, 2.0, n)
    mass /= mass.sum()
    p = dict(eps=1.0 / n, r_in=0.1 * r_out, r_out=r_out, theta=0.5, r_search=1.1 * r_out,
             n_crit=n_crit, n_leaf=16, use_quadrupole=1, precision=precision)
    w = rng.normal(size=(n, 3))
    cw = rng.normal(size=n) if with_c else None
    log(f"near vjp {precision} n={n} n_crit={n_crit} r_out={r_out}")
    gp, gm = _gpu_vjp(ctx, c.pos, mass, p, w, cw)
    op, om = oracle.Tree(c.pos, mass, p).vjp(w, cw)
    _check_vjp(gp, gm, op, om, precision, "near lists")


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_vjp_alone(ctx, precision):  # noqa: F811
    """One particle: its near list is itself, so nothing has a gradient."""
    p = dict(eps=0.01, r_in=0.05, r_out=0.5, theta=0.5, r_search=0.55, n_crit=16, n_leaf=16,
             use_quadrupole=1, precision=precision)
    gp, gm = _gpu_vjp(ctx, np.array([[0.3, -0.2, 0.1]]), np.array([1.0]), p, np.ones((1, 3)),
                      np.ones(1))
    assert np.all(gp == 0.0) and np.all(gm == 0.0)


@pytest.mark.parametrize("n", [1, 17, 70])
def test_vjp_near_far_out(ctx, n):  # noqa: F811
    """Near lists (FP64) of a cluster whose coordinates are of the size of 1e18, without
    softening, one particle at a round place: lanes past a list's end take no part."""
    c = plummer(max(n, 2), 63)
    pos = c.pos[:n] * 1e17 + 1e18
    pos[0] = 1e18
    mass = np.full(n, 1.0 / n)
    p = dict(eps=0.0, r_in=1e16, r_out=1e17, theta=0.5, r_search=1.1e17, n_crit=80, n_leaf=16,
             use_quadrupole=1, precision="fp64")
    rng = np.random.default_rng(64)
    w, cw = rng.normal(size=(n, 3)), rng.normal(size=n)
    log(f"near vjp far out n={n}")
    gp, gm = _gpu_vjp(ctx, pos, mass, p, w, cw)
    op, om = oracle.Tree(pos, mass, p).vjp(w, cw)
    assert np.all(np.isfinite(gp)) and np.all(np.isfinite(gm))
    if n > 1:
        _check_vjp(gp, gm, op, om, "fp64", "far out")
