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


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_no_memory_for_the_sums(precision, monkeypatch):
    """A build whose last requests for memory (the sums of split groups among
    them) are refused one at a time either says so or gives the same forces
    with whole groups."""
    import torch
    from paper_1506_04553_amd import P3T, P3TError
    n = 1000
    c = plummer(n, 51)
    p = dict(eps=4.0 / n, r_in=0.005, r_out=0.05, theta=0.5, r_search=0.055, n_crit=64, n_leaf=16,
             use_quadrupole=1, precision=precision)
    acc, pot = oracle.Tree(c.pos, c.mass, p).force()
    real = torch.cuda.caching_allocator_alloc
    calls = [0, -1]   # requests so far, the one to refuse

    def alloc(*args):
        calls[0] += 1
        return None if calls[0] == calls[1] else real(*args)

    monkeypatch.setattr(torch.cuda, "caching_allocator_alloc", alloc)
    pos, mass = torch.from_numpy(c.pos).cuda(), torch.from_numpy(c.mass).cuda()
    ctx = P3T(0)
    ctx.build_tree(pos, mass, **p)
    ctx.close()
    total, whole = calls[0], 0
    for k in range(4):
        calls[:] = [0, total - k]
        ctx = P3T(0)
        try:
            ctx.build_tree(pos, mass, **p)
        except P3TError as e:
            log(f"refused request {total - k} of {total}: {e}")
            ctx.close()
            continue
        a, f = ctx.long_force()
        ctx.close()
        whole += 1
        assert rel_rms(a.cpu().numpy(), acc) <= TOL[precision]
        assert rel_rms(f.cpu().numpy(), pot) <= TOL[precision]
    assert whole > 0
