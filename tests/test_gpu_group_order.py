"""The launch order of the largest inputs (2^24 groups and more: the groups in their own
order, none split), forced at sizes whose groups are otherwise split or ordered by
cost: the same forces, lists and VJP, after a build, a rebuild and a release."""
import numpy as np
import pytest

from inputs import plummer
from tests.gpu_cases import log, rel_rms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n,n_crit", [(1, 16), (3000, 700), (70000, 64)])
def test_groups_in_their_own_order(monkeypatch, n, n_crit, precision):
    import torch
    from paper_1506_04553_amd import P3T
    c = plummer(max(n, 2), 71)
    rng = np.random.default_rng(72)
    pos, mass, w, cw = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (
        c.pos[:n], c.mass[:n], rng.normal(size=(n, 3)), rng.normal(size=n)))
    p = dict(eps=4.0 / max(n, 100), r_in=0.002, r_out=0.02, theta=0.5, r_search=0.022,
             n_crit=n_crit, n_leaf=16, precision=precision)
    out = []
    for generic in (False, True):
        if generic:
            monkeypatch.setenv("P3T_GROUPS_GENERIC", "1")
        ctx = P3T(0)
        monkeypatch.delenv("P3T_GROUPS_GENERIC", raising=False)
        for k in range(3):
            if k < 2:
                ctx.build_tree(pos, mass, **p)
            else:
                ctx.release_lists()
            res = [t.cpu().numpy() for t in (*ctx.long_force(), *ctx.neighbors(),
                                             *ctx.long_force_vjp(w, cw))]
            out.append(res)
        ctx.close()
    ref = out[0]
    for k, res in enumerate(out[1:]):
        errs = [rel_rms(res[q], ref[q]) for q in (0, 1, 4, 5)]
        log(f"n={n} {precision} {k}: " + " ".join(f"{e:.1e}" for e in errs))
        assert np.array_equal(res[2], ref[2]) and np.array_equal(res[3], ref[3])
        if precision == "mixed":     # one order of summation, split or not
            assert np.array_equal(res[0], ref[0]) and np.array_equal(res[1], ref[1])
        assert max(errs[:2]) <= 1e-12
        assert max(errs[2:]) <= (1e-10 if precision == "fp64" else 1e-5)
