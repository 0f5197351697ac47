"""How p3t_hermite_hard ends where it cannot finish, with components of every class
(their kernels run on several streams): an allocation that fails leaves positions,
velocities and step counts untouched, whichever it is, and the block-step limit is
reported when nothing writes the particles any more.  The same context then gives
the oracle's result."""
import ctypes as C

import numpy as np
import pytest

import oracle
from tests.gpu_cases import log
from tests.test_gpu_hermite_classes import _components

pytestmark = pytest.mark.gpu
P = dict(eps=1e-4, r_in=0.001, r_out=0.01, theta=0.5, r_search=0.011, n_crit=64, n_leaf=16)
HK = dict(dt_soft=2.0 ** -7, dt_max=2.0 ** -9, eta=0.05, eta_s=0.005, a0=1e-5)


def _case(isolated):
    rng = np.random.default_rng(11)
    pos, off, idx = _components(rng, [1101, 1024, 300, 100, 40, 20, 9, 5, 3, 2], 0,
                                isolated=isolated)
    n = len(pos)
    vel, mass = rng.normal(scale=0.02, size=(n, 3)), rng.uniform(0.5e-6, 1.5e-6, n)
    return pos, vel, mass, off, idx


def _failing_context(state):
    """A context whose allocation number state["fail_at"] fails."""
    import torch
    from paper_1506_04553_amd import P3T
    from paper_1506_04553_amd.p3t import ALLOC_FN, FREE_FN, load_library
    st = torch.cuda.current_stream(0)

    def _alloc(nbytes, _user):
        state["count"] += 1
        if state["count"] == state["fail_at"]:
            return None
        return torch.cuda.caching_allocator_alloc(int(nbytes), 0, st)

    ctx = P3T.__new__(P3T)
    ctx._L, ctx.device, ctx.stream, ctx._allocs = load_library(), 0, st, {}
    ctx._alloc_cb = ALLOC_FN(_alloc)
    ctx._free_cb = FREE_FN(lambda p, _user: torch.cuda.caching_allocator_delete(int(p)))
    h = C.c_void_p()
    assert ctx._L.p3t_create(C.byref(h), 0, C.c_void_p(st.cuda_stream), ctx._alloc_cb, ctx._free_cb,
                             None) == 0
    ctx._h, ctx.n, ctx.params, ctx.build_id = h, 0, None, 0
    return ctx


def _call(ctx, case, hk):
    """(status, positions, velocities, steps) of one call on copies of the case."""
    import torch
    from paper_1506_04553_amd.p3t import HermiteParams, _dptr, make_params
    x, v, mass, off, idx = (torch.from_numpy(a.copy()).cuda() for a in case)
    ns = torch.full((len(mass),), -7, dtype=torch.int32, device="cuda")
    p, hp = make_params(**P), HermiteParams(**{"max_block_steps": 0, **hk})
    rc = ctx._L.p3t_hermite_hard(ctx._h, len(mass), _dptr(x), _dptr(v), _dptr(mass), _dptr(off),
                                 _dptr(idx), C.byref(p), None, C.byref(hp), _dptr(ns), None)
    # on a stream that waits for no other
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        at_once = x.clone()
    side.synchronize()
    torch.cuda.synchronize()
    assert torch.equal(at_once, x)
    return rc, x.cpu().numpy(), v.cpu().numpy(), ns.cpu().numpy()


@pytest.mark.parametrize("isolated", [50, 14500])
def test_hermite_errors(isolated):
    from paper_1506_04553_amd.p3t import P3T_ELIMIT, P3T_ENOMEM, P3T_OK
    case = _case(isolated)
    pos, vel = case[:2]
    ox, ov, ons, _ = oracle.hermite(*case, P["eps"], P["r_in"], P["r_out"], **HK)
    state = dict(count=0, fail_at=0)
    ctx = _failing_context(state)
    for k in range(1, 40):
        # each failure after one success more (what was had is kept for the next call)
        state.update(count=0, fail_at=min(k, 2))
        rc, x, v, ns = _call(ctx, case, HK)
        log(f"n {len(pos)}: call {k}: status {rc} after {state['count']} allocations")
        if rc == P3T_OK:
            break
        assert rc == P3T_ENOMEM
        assert np.array_equal(x, pos) and np.array_equal(v, vel) and np.all(ns == -7)
    assert rc == P3T_OK and k > 3
    state["fail_at"] = 0
    rc = _call(ctx, case, {**HK, "max_block_steps": 1})[0]
    assert rc == P3T_ELIMIT
    rc, x, v, ns = _call(ctx, case, HK)
    ctx.close()
    assert rc == P3T_OK
    assert np.array_equal(ns, ons) and np.array_equal(x, ox) and np.array_equal(v, ov)
