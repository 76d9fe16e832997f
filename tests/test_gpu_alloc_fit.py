"""Requests that fit are served in full: into holes of several densities, under
every search and type policy, at the request lengths of small and large creations
(64, 256 and 1,024 objects per wavefront), and where nothing is to spare; a request
for more takes what room there is."""
import pytest

pytestmark = pytest.mark.gpu

import numpy as np  # noqa: E402
import oracle  # noqa: E402
import torch  # noqa: E402
from paper_1809_07444_amd import _capi as C  # noqa: E402
from paper_1809_07444_amd import apps  # noqa: E402
from paper_1809_07444_amd.heap import Heap  # noqa: E402
from synth import workloads as W  # noqa: E402


def holes(blocks, capacity, every, search=C.SEARCH_HASHED, policy=C.POLICY_DENSE, width=64, spare=0):
    """A heap whose blocks are full but for every `every`-th object (runs of 4096 of 8192: 0)."""
    h = Heap(blocks + spare, capacity, types=((4, 4),), bitmap_width=width)
    h.set_search(search)
    objs = h.alloc_n(0, blocks * capacity)
    assert int((objs == -1).sum()) == 0
    i = torch.arange(objs.numel(), device="cuda")
    gone = (i % every == 0) if every else ((i >> 12) & 1 == 0)
    h.free_n(objs[gone].contiguous())
    h.set_type_policy(0, policy)
    return h, objs[~gone], int(gone.sum())


@pytest.mark.parametrize("search", [C.SEARCH_HASHED, C.SEARCH_LOWEST, C.SEARCH_XCD])
@pytest.mark.parametrize("capacity", [64, 32])
@pytest.mark.parametrize("blocks,every", [(1 << 13, 2), (1 << 14, 3), (1 << 14, 0), (1 << 17, 16), (1 << 17, 0), (1 << 18, 64),
                                          (1 << 18, 3)])
def test_nine_tenths_of_the_holes(blocks, every, capacity, search):
    h, left, room = holes(blocks, capacity, every, search)
    n = room * 9 // 10
    got = h.alloc_n(0, n)
    assert int((got == -1).sum()) == 0
    every_one = torch.cat([left, got])
    assert torch.unique(every_one).numel() == every_one.numel()
    st = h.stats()  # raises on any sticky flag
    assert st["live"] == [every_one.numel()]
    assert h.check() == {}


@pytest.mark.parametrize("policy", [C.POLICY_DENSE, C.POLICY_FRESH, C.POLICY_BOUNDED])
@pytest.mark.parametrize("width", [64, 32])
@pytest.mark.parametrize("every,n", [(3, 1000), (5, 200000), (3, 500000), (2, 1 << 20), (3, 1 << 21)])
def test_every_policy(every, n, policy, width):
    h, left, room = holes(-(-n * every // 64), 64, every, policy=policy, width=width, spare=16)
    got = h.alloc_n(0, n * 9 // 10)
    assert int((got == -1).sum()) == 0
    every_one = torch.cat([left, got])
    assert torch.unique(every_one).numel() == every_one.numel()
    assert h.stats()["oom"] == 0 and h.check() == {}


@pytest.mark.parametrize("search", [C.SEARCH_HASHED, C.SEARCH_XCD])
@pytest.mark.parametrize("blocks,every", [(16, 2), (1000, 3), (1 << 14, 2), (1 << 16, 3), (1 << 17, 0)])
def test_more_than_the_room(blocks, every, search):
    h, left, room = holes(blocks, 64, every, search)
    got = h.alloc_n(0, room + 5000)
    got = got[got != -1]
    st = h.stats(raise_sticky=False)
    assert st["oom"] == 1 and got.numel() == room
    assert torch.unique(torch.cat([left, got])).numel() == blocks * 64
    h.free_n(got)
    assert h.stats(raise_sticky=False)["live"] == [left.numel()] and set(h.check()) == {"sticky"}


# Three blocks per 64 cells is what serving reserves for a world (3,072 and 768 here).
@pytest.mark.parametrize("side,blocks,capacity", [(256, 3072, 64), (256, 5500, 32), (128, 768, 64), (1024, 45000, 64)])
def test_a_game_of_life_in_its_budget(side, blocks, capacity):
    g = W.gol_grid(side, side, seed=1, threshold24=1 << 22)
    want = oracle.gol_run(g, 20)[0]
    for _ in range(4):
        gol = apps.GameOfLife([g], capacity=capacity, num_blocks=blocks)
        gol.init()
        gol.step(20)
        assert gol.heap.stats()["oom"] == 0
        assert np.array_equal(gol.read()[0], want)
        gol.close()
