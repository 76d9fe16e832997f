"""Sugarscape readout of worlds that share a heap, in one launch over cells and
heap and, for large worlds, in two: every capacity and container width, heaps of
few units of blocks to many more than the launch has wavefronts, a retired
world's slot taken again, against the oracle; a readout enumerates nothing."""
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

R = W.SUGAR_RULES


class Pool:
    def __init__(self, blocks, capacity, width, worlds, arena):
        self.heap = Heap(blocks, capacity, apps.SUGAR_TYPE, bitmap_width=width)
        self.lib = self.heap.lib
        nbytes = int(self.lib.dsoar_sugarpool_bytes(worlds, arena))
        self.buf = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        rules = C.SugarRules(R["max_age"], R["repro_min"], R["fertile_min"], R["fertile_max"], 0)
        p = ctypes.c_void_p()
        C.check(self.lib.dsoar_sugarpool_create(self.heap.h, worlds, arena, ctypes.byref(rules), self.buf.data_ptr(),
                                                nbytes, ctypes.byref(p)), "create")
        self.p = p

    def admit(self, slot, off, inp):
        dev = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in
               (inp.sugar, inp.cap, inp.occ, inp.a_sugar, inp.a_metab, inp.a_vision, inp.a_age)]
        C.check(self.lib.dsoar_sugar_admit(self.p, slot, off, inp.side, inp.seed, 0, *[t.data_ptr() for t in dev],
                                           self.heap._s()), "admit")
        torch.cuda.synchronize()

    def step(self, n):
        C.check(self.lib.dsoar_sugar_step(self.p, n, C.DO_PERSISTENT, self.heap._s()), "step")

    def check(self, slot, inp, steps):
        n = inp.side * inp.side
        # Whatever was in the buffers is overwritten, cells without agents with zeros.
        outs = [torch.full((n,), 77, dtype=dt, device="cuda") for dt in
                (torch.int32, torch.uint8, torch.int32, torch.int32, torch.int32, torch.int32)]
        moves = ctypes.c_uint64()
        C.check(self.lib.dsoar_sugar_read_world(self.p, slot, *[t.data_ptr() for t in outs], ctypes.byref(moves),
                                                self.heap._s()), "read")
        torch.cuda.synchronize()
        ref = oracle.sugar_run(oracle.SugarState(inp.side, inp.sugar, inp.cap, inp.occ, inp.a_sugar, inp.a_metab,
                                                 inp.a_vision, inp.a_age), steps, inp.seed, R)
        m = ref.occ.astype(bool)
        want = [ref.sugar, ref.occ] + [np.where(m, getattr(ref, f), 0) for f in ("a_sugar", "a_metab", "a_vision", "a_age")]
        for a, b in zip(outs, want):
            assert np.array_equal(a.cpu().numpy(), b)
        assert int(moves.value) == ref.moves


# Units are 4 blocks; a launch has at most 8,192 wavefronts at 256 CUs.
@pytest.mark.parametrize("blocks,capacity,width", [(64, 64, 64), (80, 64, 32), (129, 32, 64), (200, 0, 32), (4099, 64, 64),
                                                   (40000, 64, 32), (1 << 19, 64, 64)])
def test_worlds_in_one_heap(blocks, capacity, width):
    sides = [1, 5, 16, 33]
    inputs = [W.sugar_inputs(s, (s * s + 2) // 3, seed=s) for s in sides]
    offs = np.cumsum([3] + [s * s + 1 for s in sides])
    pool = Pool(blocks, capacity, width, 5, int(offs[-1]) + 400)
    for w, (inp, off) in enumerate(zip(inputs, offs)):
        pool.admit(w, int(off), inp)
    for w, inp in enumerate(inputs):
        pool.check(w, inp, 0)
    pool.step(9)
    for w, inp in enumerate(inputs):
        pool.check(w, inp, 9)
    C.check(pool.lib.dsoar_sugar_retire(pool.p, 2, pool.heap._s()), "retire")
    again = W.sugar_inputs(16, 100, seed=77)
    pool.admit(2, int(offs[2]), again)
    pool.step(4)
    pool.check(2, again, 4)
    pool.check(3, inputs[3], 13)
    assert pool.heap.check() == {}


# 512^2 cells are the fewest that are read in two launches.
@pytest.mark.parametrize("capacity", [64, 32])
@pytest.mark.parametrize("side,fill", [(128, 0.0), (128, 1.0), (511, 0.3), (512, 0.0), (512, 1.0), (513, 0.3)])
def test_large_worlds_full_and_empty_ones(side, fill, capacity):
    inp, other = W.sugar_inputs(side, int(side * side * fill), seed=3), W.sugar_inputs(20, 150, seed=4)
    pool = Pool(side * side // capacity + 300, capacity, 64, 2, side * side + 400)
    pool.admit(1, side * side, other)
    pool.admit(0, 0, inp)
    for steps in (0, 2):
        pool.step(steps)
        pool.check(0, inp, steps)
        pool.check(1, other, steps)


def test_a_readout_enumerates_nothing():
    sim = apps.Sugarscape(W.sugar_inputs(40, 300, seed=1), R)
    sim.init()
    sim.step(3)
    before = sim.heap.stats()
    sim.heap.set_timing(True)
    sim.heap.timing()
    sim.read()
    assert set(sim.heap.timing()) <= {"sugar_read"}
    assert sim.heap.stats() == before
