"""A build allocates what its route reads: no histograms where the keys are ranked, no
scanned block counts where the blocks add up each other's."""
import pytest

from inputs import plummer
from tests.gpu_cases import log
from tests.test_zz_no_alloc import CountingContext, _build

pytestmark = pytest.mark.gpu


def _allocations(n):
    import torch
    c = plummer(n, 81)
    cx = CountingContext()
    try:
        _build(cx, torch.from_numpy(c.pos).cuda(), torch.from_numpy(c.mass).cuda(), "fp64")
        return cx.allocs
    finally:
        cx.close()


def test_allocations_by_route():
    n = {k: _allocations(k) for k in (8192, 8193, 12288, 12289, 24576, 24577)}
    log(str(n))
    # ranked in one launch; after it the box's records, second keys and indices, and the
    # packed particles
    assert n[8193] == n[8192] + 4 and n[12288] == n[8193]
    # the scan of the block counts from 49 blocks of 256 on
    assert n[12289] == n[12288] + 1 and n[24576] == n[12289]
    # two histograms and their totals
    assert n[24577] == n[24576] + 3
