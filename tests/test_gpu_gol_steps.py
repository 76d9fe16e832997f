"""Game of Life with every cell alone (eight Candidates per live cell: more
than a wavefront's queue holds), in passes of one and of two list entries, at
every block capacity and across odd numbers of generations per call, against
the oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
from paper_1809_07444_amd import _capi as C  # noqa: E402
from paper_1809_07444_amd import apps  # noqa: E402
from synth import workloads as W  # noqa: E402

GRAPH = C.DO_PERSISTENT | C.GRAPH


def run(grids, split, flags=GRAPH, capacity=64, launch=None, width=64):
    gol = apps.GameOfLife(grids, capacity=capacity, bitmap_width=width)
    if launch:
        gol.heap.set_launch(*launch)
    for again in range(2):  # the second start finds the other plane current
        gol.init()
        want = [np.ascontiguousarray(g) for g in grids]
        for k in split:
            gol.step(k, flags)
            want = [oracle.gol_run(w, k)[0] for w in want]
            for a, b in zip(gol.read(), want):
                assert np.array_equal(a, b), (again, k)
        assert gol.heap.check() == {}


def spread(n, step):
    g = np.zeros((n, n), np.uint8)
    g[::step, ::step] = 1
    return g


# 64 lanes x 8 claims against a queue of 256; a launch of 64 wavefronts makes passes of two entries.
@pytest.mark.parametrize("capacity,width", [(64, 64), (64, 32), (32, 64), (0, 64)])
@pytest.mark.parametrize("launch", [None, (64, 1), (1024, 2)])
def test_more_claims_than_the_queue_holds(capacity, width, launch):
    g = spread(192, 3)
    g[::6, 1::6] = 1  # some pairs and corners among them, so that generations go on
    run([g, spread(64, 4), W.gol_grid(150, 150, seed=3)], [1, 2, 3, 12], capacity=capacity, launch=launch, width=width)


@pytest.mark.parametrize("flags", [C.DO_PERSISTENT, C.DO_PLAIN, GRAPH])
@pytest.mark.parametrize("side", [1, 2, 3, 4, 5, 8, 33])
def test_small_tori(side, flags):
    run([W.gol_grid(side, side, seed=side, threshold24=1 << 23)], [1, 1, 3], flags=flags)


def test_births_fill_the_queue():
    # Rows of three: every generation half of the cells are born.
    g = np.zeros((256, 256), np.uint8)
    for y in range(1, 256, 4):
        for x in range(0, 252, 4):
            g[y, x:x + 3] = 1
    run([g], [1, 2, 5], launch=(64, 1))
