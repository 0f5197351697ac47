"""p3t_release_lists gives back, besides the lists, the partial sums of split groups
and the direct sums' workspace; what the next calls return is the same."""
import numpy as np
import pytest

from inputs import plummer
from tests.gpu_cases import log
from tests.test_zz_no_alloc import CountingContext, _p

pytestmark = pytest.mark.gpu
MIB = 1 << 20


class TrackingContext(CountingContext):
    """... and knows the sizes of what its allocator still holds."""

    def __init__(self):
        import torch
        self.live, alloc, delete = {}, torch.cuda.caching_allocator_alloc, \
            torch.cuda.caching_allocator_delete

        def tracked(nbytes, *a):
            ptr = alloc(nbytes, *a)
            self.live[ptr] = nbytes
            return ptr

        def untracked(ptr):
            self.live.pop(ptr)
            delete(ptr)

        self._torch, self._own = torch.cuda, (alloc, delete)
        torch.cuda.caching_allocator_alloc, torch.cuda.caching_allocator_delete = tracked, untracked
        super().__init__()

    def close(self):
        super().close()
        self._torch.caching_allocator_alloc, self._torch.caching_allocator_delete = self._own


def test_release_gives_back_the_workspaces():
    import ctypes as C
    import torch
    from paper_1506_04553_amd import make_params
    n = 60000
    c = plummer(n, 6)
    pos, mass = torch.from_numpy(c.pos).cuda(), torch.from_numpy(c.mass).cuda()
    prm = make_params(eps=1e-3, r_in=0.002, r_out=0.02, theta=0.5, r_search=0.022, n_crit=n,
                      n_leaf=2000)
    cx = TrackingContext()
    try:
        def sums():
            f, d = (torch.full((n, 3), np.nan, dtype=torch.float64, device="cuda") for _ in range(2))
            cx.check(cx.L.p3t_long_force(cx.h, _p(f), None))
            cx.check(cx.L.p3t_direct(cx.h, n, _p(pos), _p(mass), C.byref(prm), 0, _p(d), None))
            torch.cuda.synchronize()
            return f, d
        cx.check(cx.L.p3t_build_tree(cx.h, n, _p(pos), _p(mass), C.byref(prm)))
        first = sums()
        before = sum(cx.live.values())
        cx.check(cx.L.p3t_release_lists(cx.h))
        after = sum(cx.live.values())
        log(f"{before / MIB:.0f} MiB held, {after / MIB:.0f} after the release")
        # 35 parts and more of 60000 sums of 32 bytes (64 MiB); and 30 distances of the
        # direct sums' 59 blocks, two rows of 60416 sums each, with an eighth of headroom
        # (124 MiB)
        assert before - after > 188 * MIB
        again = sums()
        assert torch.equal(first[0], again[0]) and torch.equal(first[1], again[1])
    finally:
        cx.close()
