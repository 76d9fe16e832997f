"""Merging bodies at the counts where the roots' search changes from a scan of
all ids to walks through the cells, with crowds that no walk gets through, roots
that absorb none, one and many, and bodies that died in earlier steps, against
the oracle, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
from paper_1809_07444_amd import _capi as C  # noqa: E402
from paper_1809_07444_amd import apps  # noqa: E402
from synth import workloads as W  # noqa: E402


@pytest.mark.parametrize("flags,capacity", [(C.DO_PERSISTENT | C.GRAPH, 64), (C.DO_PLAIN, 32)])
@pytest.mark.parametrize("n,box,crowd", [(16, 0.05, 0), (64, 0.1, 0), (1023, 0.8, 0), (1024, 0.8, 90), (1025, 0.8, 0),
                                         (1025, 0.8, 90), (1400, 0.3, 40)])
def test_merges(n, box, crowd, flags, capacity):
    inp = W.collide_inputs(n, seed=n + crowd, box=box)
    if crowd:  # at one point, among the others' ids
        at = slice(7, 7 + 11 * crowd, 11)
        inp.x[at], inp.y[at] = box / 3, box / 5
    sim = apps.Collisions(inp, W.COLLIDE_PARAMS, capacity=capacity)
    sim.init()
    sim.step(6, flags)
    got = sim.read()
    ref = oracle.collide_run(oracle.CollideState(inp.x, inp.y, inp.vx, inp.vy, inp.m), 6, W.COLLIDE_PARAMS)
    assert ref.merges >= max(1, crowd - 1)
    for f in ("x", "y", "vx", "vy", "m"):
        assert np.array_equal(getattr(got, f).view(np.uint32), getattr(ref, f).view(np.uint32)), f
    assert got.stats["frees"] == [ref.merges] and got.stats["live"] == [int((ref.m > 0).sum())]
    assert sim.heap.check() == {}
