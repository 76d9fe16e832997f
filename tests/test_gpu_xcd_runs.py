"""Allocation under the per-XCD search policy, and Sugarscape with its lists and
initial cells cut into eight runs, one per XCD, against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
import torch  # noqa: E402
from paper_1809_07444_amd import _capi as C  # noqa: E402
from paper_1809_07444_amd import apps  # noqa: E402
from paper_1809_07444_amd.heap import Heap  # noqa: E402
from synth import workloads as W  # noqa: E402


# Lists shorter than, equal to and just over the runs; a heap of one, two and three bitmap levels.
@pytest.mark.parametrize("capacity", [64, 32, 0])
@pytest.mark.parametrize("blocks,objects", [(16, 1), (16, 449), (64, 64 * 7), (64, 64 * 8 + 1), (5000, 64 * 4000 + 3)])
@pytest.mark.parametrize("width", [64, 32])
def test_every_object_once(blocks, objects, capacity, width):
    h = Heap(blocks * (2 if capacity == 32 else 1), capacity, types=((4, 4),), bitmap_width=width)
    h.set_search(C.SEARCH_XCD)
    objs = h.alloc_n(0, objects)
    assert int((objs == -1).sum()) == 0 and torch.unique(objs).numel() == objects
    want = torch.zeros(h.num_blocks * 64, dtype=torch.int32, device="cuda")
    want[objs.long()] = 1
    for flags in (C.DO_PERSISTENT, C.DO_PLAIN):
        for wg, per_cu in ((256, 8), (64, 1)):
            h.set_launch(wg, per_cu)
            assert torch.equal(h.visit_counts(0, flags), want)
    h.free_n(objs)
    assert int(h.visit_counts(0).sum()) == 0
    assert h.check() == {}


# Lists of no block, fewer blocks than XCDs, a few more; plain grids of any size; 32 slots per block.
@pytest.mark.parametrize("capacity", [64, 32])
@pytest.mark.parametrize("flags", [C.DO_PERSISTENT | C.GRAPH, C.DO_PLAIN])
@pytest.mark.parametrize("side,agents", [(16, 0), (16, 1), (16, 40), (97, 2000), (130, 4000)])
def test_sugarscape(side, agents, flags, capacity):
    inp = W.sugar_inputs(side, agents, seed=side)
    sim = apps.Sugarscape(inp, W.SUGAR_RULES, capacity=capacity)
    sim.heap.set_search(C.SEARCH_XCD)
    sim.init()
    sim.step(25, flags)
    got = sim.read()
    ref = oracle.SugarState(side, inp.sugar, inp.cap, inp.occ, inp.a_sugar, inp.a_metab, inp.a_vision, inp.a_age)
    ref = oracle.sugar_run(ref, 25, inp.seed, W.SUGAR_RULES)
    assert np.array_equal(got.sugar, ref.sugar) and np.array_equal(got.occ, ref.occ) and got.moves == ref.moves
    m = ref.occ.astype(bool)
    for f in ("a_sugar", "a_metab", "a_vision", "a_age"):
        assert np.array_equal(getattr(got, f)[m], getattr(ref, f)[m]), f
    assert sim.heap.check() == {}
