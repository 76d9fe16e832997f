"""Wa-Tor's byte planes (rows in groups of four), pruned lists and queued births
at the edges: sides below and beside whole groups, both block capacities,
passes of one and of two list entries, calls of one and of many steps, and the
visits that the counters report, against the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
from paper_1809_07444_amd import _capi as C  # noqa: E402
from paper_1809_07444_amd import apps  # noqa: E402
from synth import workloads as W  # noqa: E402

GRAPH = C.DO_PERSISTENT | C.GRAPH
QUICK = dict(fish_breed=1, shark_breed=2, starve=2)


def run(inp, rules, split, flags=GRAPH, capacity=64, launch=None, online=False):
    sea = apps.Wator(inp, rules, capacity=capacity)
    if launch:
        sea.heap.set_launch(*launch)
    if online:
        sea.heap.set_reclaim(True)
    sea.init(step0=3)
    ref = oracle.WatorState(inp.kind, inp.age, inp.energy)
    done, fish, sharks = 3, 0, 0
    for k in split:
        sea.step(k, flags)
        for _ in range(k):
            n, s, born = int((ref.kind == 1).sum()), int((ref.kind == 2).sum()), ref.fish_born
            ref = oracle.wator_run(ref, 1, inp.seed, rules, step0=done)
            done += 1
            fish += 2 * n + n + ref.fish_born - born  # decide, move; eaten: the newborn too
            sharks += 2 * s
        got = sea.read()
        for f in ("kind", "age", "energy"):
            assert np.array_equal(getattr(got, f), getattr(ref, f)), (f, done)
        live = [int((ref.kind == 1).sum()), int((ref.kind == 2).sum())]
        fish, sharks = fish + live[0], sharks + live[1]  # the readout's
        assert got.stats["live"] == live
        assert got.stats["frees"] == [ref.fish_eaten, ref.sharks_starved]
        assert got.stats["visits"] == [fish, sharks], done
    assert sea.heap.check() == {}
    sea.close()


@pytest.mark.parametrize("flags", [C.DO_PERSISTENT, C.DO_PLAIN, GRAPH])
@pytest.mark.parametrize("side", [1, 2, 3, 4, 5, 6, 7, 8, 33, 66])
def test_sides(side, flags):
    run(W.wator_inputs(side, seed=side, fish24=int(0.4 * (1 << 24)), shark24=int(0.2 * (1 << 24))), QUICK, [1, 1, 12],
        flags)


# Every fish breeds whenever it moves: more newborns than a wavefront's queue holds.
@pytest.mark.parametrize("launch", [(64, 1), (1024, 2)])
@pytest.mark.parametrize("capacity", [64, 32, 0])
@pytest.mark.parametrize("online", [False, True])
def test_lists_and_queues(capacity, launch, online):
    run(W.wator_inputs(190, seed=4, fish24=int(0.2 * (1 << 24)), shark24=int(0.02 * (1 << 24))), QUICK, [1, 2, 13],
        capacity=capacity, launch=launch, online=online)


def test_blocks_that_the_sharks_empty():
    # Whole blocks of fish (64 cells of a row in a block) between rows of sharks.
    side = 64
    kind = np.zeros((side, side), np.int32)
    kind[::4] = 1
    kind[1::4] = 2
    kind[3::4] = 2
    inp = W.WatorInputs(side, 7, kind, np.zeros_like(kind), np.where(kind == 2, 3, 0).astype(np.int32))
    run(inp, dict(fish_breed=50, shark_breed=50, starve=3), [4, 1, 6])
