"""Wa-Tor's initial sea with one and with four cells per lane, at the sides where
the one gives way to the other and with remainders of four cells, empty and full
seas among them, and the steps that follow, against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
from paper_1809_07444_amd import apps  # noqa: E402
from synth import workloads as W  # noqa: E402


# 724^2 is the largest sea below 2^19 cells.
@pytest.mark.parametrize("side,fish,sharks,capacity", [(1, 1.0, 0.0, 64), (15, 0.5, 0.5, 32), (16, 0.0, 0.0, 64), (33, 0.0, 1.0, 64),
                                                       (723, 0.3, 0.1, 64), (724, 0.3, 0.05, 32), (725, 0.3, 0.05, 64),
                                                       (725, 0.95, 0.05, 64), (726, 0.01, 0.01, 32), (727, 0.3, 0.3, 64)])
def test_initial_sea(side, fish, sharks, capacity):
    rng = np.random.default_rng(side)
    u = rng.random((side, side))
    kind = np.where(u < fish, 1, np.where(u < fish + sharks, 2, 0)).astype(np.int32)
    age = np.where(kind > 0, rng.integers(0, 3, kind.shape), 0).astype(np.int32)
    energy = np.where(kind == 2, rng.integers(1, 4, kind.shape), 0).astype(np.int32)
    inp = W.WatorInputs(side, 5, kind, age, energy)
    sea = apps.Wator(inp, W.WATOR_RULES, capacity=capacity)
    sea.init(step0=2)
    ref = oracle.WatorState(kind, age, energy)
    for steps in (0, 3):
        sea.step(steps)
        ref = oracle.wator_run(ref, steps, inp.seed, W.WATOR_RULES, step0=2) if steps else ref
        got = sea.read()
        for f in ("kind", "age", "energy"):
            assert np.array_equal(getattr(got, f), getattr(ref, f)), (f, steps)
        assert got.stats["live"] == [int((ref.kind == 1).sum()), int((ref.kind == 2).sum())]
    assert sea.heap.check() == {}
