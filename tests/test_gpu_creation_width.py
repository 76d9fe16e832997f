"""Creations at the sizes where a lane's share of a request changes (one, four,
sixteen objects), with remainders, on empty heaps, on heaps with holes and on
heaps too small for them: every object once, no slot twice, misses reported."""
import pytest

pytestmark = pytest.mark.gpu

import torch  # noqa: E402
from paper_1809_07444_amd import _capi as C  # noqa: E402
from paper_1809_07444_amd.heap import Heap  # noqa: E402

SIZES = [1, 63, 65, (1 << 18) - 1, 1 << 18, (1 << 18) + 1, (1 << 20) - 1, 1 << 20, (1 << 20) + 1023]


@pytest.mark.parametrize("policy", [C.POLICY_DENSE, C.POLICY_FRESH, C.POLICY_BOUNDED])
@pytest.mark.parametrize("n", SIZES)
def test_holes_and_full_heaps(n, policy):
    blocks = -(-n // 64) + 64
    h = Heap(blocks, 64, types=((4, 4),))
    h.set_type_policy(0, policy)
    objs = h.alloc_n(0, n)
    assert int((objs == -1).sum()) == 0 and torch.unique(objs).numel() == n
    gone = torch.arange(n, device="cuda") % 3 == 0
    h.free_n(objs[gone].contiguous())
    left = objs[~gone]
    room = blocks * 64 - left.numel()
    again = h.alloc_n(0, room // 2)  # into the holes
    assert int((again == -1).sum()) == 0
    more = h.alloc_n(0, n)  # more than fits
    got = more[more != -1]
    every = torch.cat([left, again, got])
    assert torch.unique(every).numel() == every.numel() <= blocks * 64
    st = h.stats(raise_sticky=False)
    assert st["live"] == [every.numel()] and st["oom"] == (1 if got.numel() < n else 0)


@pytest.mark.parametrize("n", SIZES)
def test_micro_objects_in_order(n):
    h = Heap(-(-n // 32) + 64, 64, types=((4, 4, 4),))
    xs = torch.arange(n, device="cuda", dtype=torch.float32)
    C.check(h.lib.dsoar_micro_init(h.h, 0, n, xs.data_ptr(), (-xs).contiguous().data_ptr(), h._s()), "dsoar_micro_init")
    (x, px), (v, pv) = h.gather(0, 0, 1, n), h.gather(0, 0, 2, n)
    assert bool(px.bool().all()) and bool(pv.bool().all())
    assert torch.equal(x.view(torch.float32), xs) and torch.equal(v.view(torch.float32), -xs)
    assert h.check() == {}
