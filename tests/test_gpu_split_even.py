"""Groups of about the same cost, which mixed precision leaves whole from 256 of them on
(fewer are split): forces, potentials and gradients on either side, against the oracle."""
import numpy as np
import pytest

import oracle
from tests.gpu_cases import ROW_TOL, gpu_run, log, rel_rms, row_errors

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("places", [255, 256, 400])
def test_even_groups(places):
    import torch
    from paper_1506_04553_amd import P3T
    rng = np.random.default_rng(places)
    copies = 20                      # more than n_crit: each place is a leaf and a group
    pos = np.repeat(rng.uniform(-1, 1, (places, 3)), copies, axis=0)
    n = len(pos)
    mass = rng.uniform(0.5, 2.0, n) / n
    p = dict(eps=4.0 / n, r_in=1e-5, r_out=1e-4, theta=0.5, r_search=1.1e-4, n_crit=16, n_leaf=16,
             precision="mixed")
    ctx = P3T(0)
    g = gpu_run(ctx, pos, mass, p, want_neighbors=False, want_arrays=False)
    assert g["stats"]["n_groups"] == places
    log(f"{places} even groups")
    w, c = rng.normal(size=(n, 3)), rng.normal(size=n)
    gpos, gmass = (t.cpu().numpy() for t in ctx.long_force_vjp(torch.from_numpy(w).cuda(),
                                                              torch.from_numpy(c).cuda()))
    ctx.close()
    t = oracle.Tree(pos, mass, p)
    acc, pot = t.force()
    opos, omass = t.vjp(w, c)
    assert rel_rms(g["acc"], acc) <= 1e-4 and rel_rms(g["pot"], pot) <= 1e-4
    assert row_errors(g["acc"], acc) <= ROW_TOL["mixed"]
    assert row_errors(g["pot"], pot) <= ROW_TOL["mixed"]
    assert rel_rms(gpos, opos) <= 1e-4 and rel_rms(gmass, omass) <= 1e-4
