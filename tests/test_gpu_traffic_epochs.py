"""Traffic over more steps than the road planes' epochs go round in (4,094),
with old words left behind by cars at every age, against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
from paper_1809_07444_amd import _capi as C  # noqa: E402
from paper_1809_07444_amd import apps  # noqa: E402
from synth import workloads as W  # noqa: E402


# Sparse roads keep words of many epochs; 1 x 1, odd cell counts and fewer words than sweep parts.
@pytest.mark.parametrize("roads,length,p_in,capacity", [(1, 1, 1 << 23, 64), (3, 51, 1 << 10, 64), (7, 333, 1 << 14, 32),
                                                        (40, 100, 1 << 16, 64)])
def test_epochs_go_round(roads, length, p_in, capacity):
    inp = W.traffic_inputs(roads, length, seed=roads)
    rules = dict(vmax=5, p_slow24=1 << 22, p_in24=p_in)
    sim = apps.Traffic(inp, rules, capacity=capacity)
    sim.init()
    vel, done = inp.vel, 0
    for k in (4090, 3, 1, 1, 2, 4100, 1000):
        sim.step(k, C.DO_PERSISTENT | C.GRAPH)
        vel = oracle.traffic_run(vel, k, inp.seed, rules, step0=done).vel
        done += k
        assert np.array_equal(sim.read(), vel), f"differs after {done} steps"
    assert sim.heap.check() == {}

