"""Traffic in heaps whose room for entering cars is what the leaving cars of the
same step free: the cars then enter after the others have moved, against the
oracle."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
import torch  # noqa: E402
from paper_1809_07444_amd import _capi as C  # noqa: E402
from paper_1809_07444_amd import apps  # noqa: E402
from paper_1809_07444_amd.heap import Heap  # noqa: E402
from synth import workloads as W  # noqa: E402


# Roads of one cell: every car leaves in every step and another enters.  A
# quarter of the heap is spare, or as many slots as cars (enough for both at once).
# (Dense policy: under the others the blocks that the leaving cars empty, which
# are free at the next enumeration only, are looked up late.)
@pytest.mark.parametrize("flags", [C.DO_PERSISTENT, C.DO_PERSISTENT | C.GRAPH, C.DO_PLAIN])
@pytest.mark.parametrize("roads,capacity,room", [(1 << 20, 64, 1.25), (1 << 20, 32, 1.25), (1000, 64, 1.3), (1 << 16, 64, 2.0),
                                                 ((1 << 16) + 1, 64, 2.0)])
def test_every_car_replaced(roads, capacity, room, flags):
    inp = W.traffic_inputs(roads, 1, seed=1)
    inp.vel[:] = 0
    rules = dict(vmax=5, p_slow24=0, p_in24=1 << 24)
    sim = apps.Traffic(inp, rules, capacity=capacity, num_blocks=int(roads * room) // capacity)
    sim.heap.set_type_policy(0, C.POLICY_DENSE)
    sim.init()
    sim.step(5, flags)
    got = sim.read()
    st = sim.heap.stats(raise_sticky=False)
    assert st["oom"] == 0 and st["live"] == [roads]
    assert np.array_equal(got, oracle.traffic_run(inp.vel, 5, inp.seed, rules, step0=0).vel)
    assert st["visits"] == [2 * 5 * roads]
    assert sim.heap.check() == {}


def test_another_type_holds_blocks():
    # Roads of eight cells and a heap of twice the cells, but for the blocks that a second type has taken.
    roads, length = 4096, 8
    inp = W.traffic_inputs(roads, length, seed=3)
    rules = dict(vmax=5, p_slow24=1 << 20, p_in24=1 << 24)
    sim = apps.Traffic(inp, rules)
    heap = Heap(2 * roads * length // 64, 64, [(4, 4, 4), (4, 4)], stream=sim.stream)
    t = ctypes.c_void_p()
    C.check(sim.lib.dsoar_traffic_create(heap.h, roads, length, ctypes.byref(sim.rules), sim.buf.data_ptr(),
                                         int(sim.lib.dsoar_traffic_bytes(roads, length)), ctypes.byref(t)), "create")
    sim.close()
    sim.t, sim.heap = t, heap
    sim.init()
    heap.alloc_n(1, 64 * (heap.num_blocks // 2 - 64))
    sim.step(20)
    vel = oracle.traffic_run(inp.vel, 20, inp.seed, rules, step0=0).vel
    assert np.array_equal(sim.read(), vel)
    assert heap.stats(raise_sticky=False)["oom"] == 0
    torch.cuda.synchronize()
    assert heap.check() == {}


# Sparse and dense roads, one launch and two, of whole and odd sizes.
@pytest.mark.parametrize("roads,length,blocks", [(300, 40, None), (300, 40, 192), (65, 7, 8), (65, 7, None), (1, 100, 64)])
def test_both_forms(roads, length, blocks):
    inp = W.traffic_inputs(roads, length, seed=5)
    rules = dict(vmax=5, p_slow24=1 << 22, p_in24=1 << 23)
    sim = apps.Traffic(inp, rules, num_blocks=blocks)
    sim.init()
    vel, done = inp.vel, 0
    for k in (1, 2, 17):
        sim.step(k)
        vel = oracle.traffic_run(vel, k, inp.seed, rules, step0=done).vel
        done += k
        assert np.array_equal(sim.read(), vel)
    assert sim.heap.check() == {}
