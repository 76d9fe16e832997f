"""Sugarscape admission with one cell and with four rows of cells per lane, at the
sides where the one gives way to the other and with every remainder of four
rows, and the steps that follow, against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
from paper_1809_07444_amd import _capi as C  # noqa: E402
from paper_1809_07444_amd import apps  # noqa: E402
from synth import workloads as W  # noqa: E402


# 362^2 is the largest below 2^17 cells.
@pytest.mark.parametrize("capacity", [64, 32])
@pytest.mark.parametrize("side,fill", [(9, 1.0), (361, 0.2), (362, 1.0), (363, 1.0), (364, 0.2), (365, 0.5), (366, 0.02)])
def test_admission(side, fill, capacity):
    inp = W.sugar_inputs(side, int(side * side * fill), seed=side)
    sim = apps.Sugarscape(inp, W.SUGAR_RULES, capacity=capacity)
    sim.init()
    ref = oracle.SugarState(side, inp.sugar, inp.cap, inp.occ, inp.a_sugar, inp.a_metab, inp.a_vision, inp.a_age)
    done = 0
    for k in (0, 6):
        sim.step(k, C.DO_PERSISTENT)
        done += k
        got, want = sim.read(), oracle.sugar_run(ref, done, inp.seed, W.SUGAR_RULES)
        assert np.array_equal(got.sugar, want.sugar) and np.array_equal(got.occ, want.occ) and got.moves == want.moves
        m = want.occ.astype(bool)
        for f in ("a_sugar", "a_metab", "a_vision", "a_age"):
            assert np.array_equal(getattr(got, f)[m], getattr(want, f)[m]), f
        assert got.stats["oom"] == 0
    assert sim.heap.check() == {}
