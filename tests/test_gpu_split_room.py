"""The partial sums of split groups within their bound of 256 MiB (and an eighth of
headroom): long lists of many groups in FP32, of which only the costliest can be cut
into parts, and one group of many rounds in FP64, which takes no more than its parts
need."""
import ctypes as C

import numpy as np
import pytest

import oracle
from inputs import plummer
from tests.gpu_cases import ROW_TOL, log, rel_rms, row_errors

pytestmark = pytest.mark.gpu
MIB = 1 << 20


def _run(c, p, direct=False):
    """Forces of a build in a new context, its groups and its allocations' sizes."""
    import torch
    from paper_1506_04553_amd import P3T
    from paper_1506_04553_amd.p3t import ALLOC_FN, FREE_FN, load_library
    st, sizes = torch.cuda.current_stream(0), []

    def _alloc(nbytes, _user):
        sizes.append(int(nbytes))
        return torch.cuda.caching_allocator_alloc(int(nbytes), 0, st)

    ctx = P3T.__new__(P3T)
    ctx._L, ctx.device, ctx.stream, ctx._allocs = load_library(), 0, st, {}
    ctx._alloc_cb = ALLOC_FN(_alloc)
    ctx._free_cb = FREE_FN(lambda q, _user: torch.cuda.caching_allocator_delete(int(q)))
    h = C.c_void_p()
    assert ctx._L.p3t_create(C.byref(h), 0, C.c_void_p(st.cuda_stream), ctx._alloc_cb, ctx._free_cb,
                             None) == 0
    ctx._h, ctx.n, ctx.params, ctx.build_id = h, 0, None, 0
    pos, mass = torch.from_numpy(c.pos).cuda(), torch.from_numpy(c.mass).cuda()
    ctx.build_tree(pos, mass, **p)
    acc, pot = ctx.long_force()
    groups, most = ctx.stats()["n_groups"], list(sizes)
    ref = ctx.direct(pos, mass, "soft", **p) if direct else (acc, pot)
    out = [t.cpu().numpy() for t in (acc, pot, *ref)]
    ctx.close()
    return out, groups, most


def test_room_for_the_costliest_groups():
    n = 40000
    c = plummer(n, 5)
    p = dict(eps=1e-3, r_in=0.002, r_out=0.02, theta=0.0, r_search=0.022, n_crit=256, n_leaf=64,
             precision="mixed")
    (acc, pot, _, _), groups, sizes = _run(c, p)
    log(f"{groups} groups, largest allocation {max(sizes) / MIB:.0f} MiB")
    # all groups' partial sums would take 335 MiB; the walk's stacks take 115
    assert 150 * MIB < max(sizes) <= 289 * MIB and groups <= 1280
    again = _run(c, p)[0]
    assert np.array_equal(acc, again[0]) and np.array_equal(pot, again[1])
    racc, rpot = oracle.Tree(c.pos, c.mass, p).force()
    assert rel_rms(acc, racc) <= 1e-4 and rel_rms(pot, rpot) <= 1e-4
    assert row_errors(acc, racc) <= ROW_TOL["mixed"] and row_errors(pot, rpot) <= ROW_TOL["mixed"]


def test_room_of_one_group_in_rounds():
    n = 60000
    c = plummer(n, 6)
    p = dict(eps=1e-3, r_in=0.002, r_out=0.02, theta=0.5, r_search=0.022, n_crit=n, n_leaf=2000)
    (acc, pot, dacc, dpot), groups, sizes = _run(c, p, direct=True)
    log(f"{groups} group, largest allocation {max(sizes) / MIB:.0f} MiB")
    # at most 4096 parts and as many rounded up, of the 512 members of a round, and one
    # sum of each member: less than 2 x 64 MiB
    assert groups == 1 and max(sizes) < 150 * MIB
    assert rel_rms(acc, dacc) <= 1e-12 and rel_rms(pot, dpot) <= 1e-12
