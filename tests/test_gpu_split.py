"""Groups whose interactions are split over several blocks.

With few groups every one is split: into parts of its lists and, when its
members take more than eight virtual wavefronts, into rounds.  Checked against
the oracle on the same tree: group sizes around the 64 lanes of a wavefront
(one lane per member, then several slices per member), groups of more than 512
members (several rounds), lists shorter than one 256-entry unit and empty ones,
and leaves of one member.  Tolerances: those of the whole-group kernel (the
split kernel evaluates the same terms).
"""
import numpy as np
import pytest

import oracle
from inputs import plummer
from tests.gpu_cases import ROW_TOL, gpu_run, log, rel_rms, row_errors

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "mixed": 1e-4}


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n,n_crit,n_leaf,theta,quad", [
    (65, 64, 16, 0.5, 1), (1000, 64, 16, 0.5, 1), (1500, 61, 8, 0.7, 0), (3000, 1, 1, 0.6, 1),
    (5000, 700, 16, 0.4, 1), (2000, 2000, 16, 0.5, 1), (1300, 130, 16, 0.0, 1)])
def test_split_groups_match_oracle(n, n_crit, n_leaf, theta, quad, precision):
    import torch
    from paper_1506_04553_amd import P3T
    assert torch.cuda.is_available()
    c = plummer(n, 51)
    mass = np.random.default_rng(52).uniform(0.5, 2.0, n)
    mass /= mass.sum()
    p = dict(eps=4.0 / n, r_in=0.005, r_out=0.05, theta=theta, r_search=0.055, n_crit=n_crit,
             n_leaf=n_leaf, use_quadrupole=quad, precision=precision)
    log(f"split n={n} n_crit={n_crit} theta={theta} {precision}")
    ctx = P3T(0)
    g = gpu_run(ctx, c.pos, mass, p, want_neighbors=False, want_arrays=False)
    again = gpu_run(ctx, c.pos, mass, p, want_neighbors=False, want_arrays=False)
    ctx.close()
    acc, pot = oracle.Tree(c.pos, mass, p).force()
    assert rel_rms(g["acc"], acc) <= TOL[precision] and rel_rms(g["pot"], pot) <= TOL[precision]
    assert row_errors(g["acc"], acc) <= ROW_TOL[precision]
    assert row_errors(g["pot"], pot) <= ROW_TOL[precision]
    # a second build (lists in reserved segments) and a fixed summation order
    assert np.array_equal(again["acc"], g["acc"]) and np.array_equal(again["pot"], g["pot"])
