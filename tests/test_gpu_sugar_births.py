"""Sugarscape births by the queue: nearly every agent with a free neighbour has
a child, on lists of one and of two entries per pass, in one run and in eight,
at the sides below and beside the groups of four rows, against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
from paper_1809_07444_amd import _capi as C  # noqa: E402
from paper_1809_07444_amd import apps  # noqa: E402
from synth import workloads as W  # noqa: E402

RULES = dict(W.SUGAR_RULES, repro_min=2, fertile_min=0, fertile_max=W.SUGAR_RULES["max_age"])


@pytest.mark.parametrize("search", [C.SEARCH_HASHED, C.SEARCH_XCD])
@pytest.mark.parametrize("capacity", [64, 32])
@pytest.mark.parametrize("side,agents,launch", [(1, 1, None), (2, 1, None), (3, 2, None), (5, 3, None), (6, 9, None),
                                                (7, 12, None), (66, 700, (64, 1)), (301, 40000, (64, 1)),
                                                (301, 40000, (1024, 2))])
def test_many_births(side, agents, launch, capacity, search):
    inp = W.sugar_inputs(side, agents, seed=side)
    sim = apps.Sugarscape(inp, RULES, capacity=capacity)
    sim.heap.set_search(search)
    if launch:
        sim.heap.set_launch(*launch)
    sim.init()
    ref = oracle.SugarState(side, inp.sugar, inp.cap, inp.occ, inp.a_sugar, inp.a_metab, inp.a_vision, inp.a_age)
    done = 0
    for k in (1, 4):
        sim.step(k, C.DO_PERSISTENT)
        done += k
        got = sim.read()
        want = oracle.sugar_run(ref, done, inp.seed, RULES)
        assert np.array_equal(got.sugar, want.sugar) and np.array_equal(got.occ, want.occ) and got.moves == want.moves
        m = want.occ.astype(bool)
        for f in ("a_sugar", "a_metab", "a_vision", "a_age"):
            assert np.array_equal(getattr(got, f)[m], getattr(want, f)[m]), f
    assert sim.heap.check() == {}
