"""Force do-all at the edges of its tiles and of its arithmetic's two forms,
against the oracle: every operation is rounded once in the oracle's order, so
the results are equal bit for bit (NaN wherever the oracle has NaN)."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
from paper_1809_07444_amd import _capi as C  # noqa: E402
from paper_1809_07444_amd import apps  # noqa: E402
from synth import workloads as W  # noqa: E402

FIELDS = ("x", "y", "vx", "vy", "m")


def same(inp, params, steps, capacity=64, flags=C.DO_PERSISTENT, least=False):
    sim = apps.Collisions(inp, params, capacity=capacity)
    if least:  # the smallest buffer: no table of cells
        sim.close()
        c = ctypes.c_void_p()
        C.check(sim.lib.dsoar_collide_create(sim.heap.h, inp.n, ctypes.byref(sim.params), sim.buf.data_ptr(),
                                             sim.lib.dsoar_collide_bytes(inp.n), ctypes.byref(c)), "create")
        sim.c = c
    sim.init()
    sim.step(steps, flags)
    ref = oracle.collide_run(oracle.CollideState(inp.x, inp.y, inp.vx, inp.vy, inp.m), steps, params)
    got = sim.read()
    for f in FIELDS:
        a, b = getattr(got, f), getattr(ref, f)
        nan = np.isnan(b)
        assert np.array_equal(np.isnan(a), nan), f
        assert np.array_equal(a.view(np.uint32)[~nan], b.view(np.uint32)[~nan]), f
    assert got.stats["frees"] == [ref.merges] and got.stats["live"] == [int((ref.m > 0).sum())]
    assert sim.heap.check() == {}
    return ref


# Groups of 32 bodies, tiles of 128 ids.
@pytest.mark.parametrize("capacity", [64, 32])
@pytest.mark.parametrize("n", [1, 31, 32, 33, 64, 65, 127, 128, 129, 257, 1025])
def test_tile_edges(n, capacity):
    same(W.collide_inputs(n, seed=n, box=4.0), dict(dt=0.01, eps2=0.01, r2_merge=0.0), 3, capacity,
         C.DO_PLAIN if n == 65 else C.DO_PERSISTENT)


# One body of 300 (in the second tile's first part) outside what the short form
# of the scale takes, or eps2 itself outside.
@pytest.mark.parametrize("field,value", [("x", 2.0 ** 18), ("y", -(2.0 ** 18) - 1.0), ("x", 3.0e38), ("y", np.inf),
                                         ("x", np.nan), ("m", 2.0 ** -41), ("m", 2.0 ** 41), ("m", 2.0 ** 40),
                                         ("m", float.fromhex("0x1.ccccc4p-9")), ("m", np.inf), ("eps2", 2.0 ** -41),
                                         ("eps2", 2.0 ** -40), ("eps2", 2.0 ** 39)])
def test_range_edges(field, value):
    inp = W.collide_inputs(300, seed=9, box=4.0)
    params = dict(dt=0.01, eps2=0.01, r2_merge=0.0)
    if field == "eps2":
        params["eps2"] = value
    else:
        getattr(inp, field)[130] = value
    same(inp, params, 2)


def test_the_quotient_left_to_the_general_form():
    # r2 = 0x1.fffffap+1 = eps2 (both bodies at one point): m / (r2 sqrt(r2)) for the mass of that mantissa.
    eps2, m = float.fromhex("0x1.fffffap+1"), float.fromhex("0x1.ccccc4p+0")
    n = 40
    inp = W.collide_inputs(n, seed=2, box=1.0)
    inp.x[:], inp.y[:] = 0.5, 0.25
    inp.x[7] = np.nextafter(np.float32(0.5), np.float32(1))
    inp.m[:] = m
    same(inp, dict(dt=1.0, eps2=eps2, r2_merge=0.0), 1)


# Merge phases.  Cells: a few bodies near each other, crowds longer than a
# walk (one point, or everything in one cell), bodies outside the cells' range,
# radii that the cells do not serve.
@pytest.mark.parametrize("n,box,r2,capacity", [
    (1, 1.0, 1e-4, 64), (2, 0.001, 1e-4, 64), (500, 0.4, 1e-4, 64), (500, 0.4, 1e-4, 32), (3000, 0.4, 1e-4, 64),
    (200, 0.0, 1e-4, 64), (300, 0.5, 0.25, 64), (200, 1.0, 2.0 ** -61, 64), (200, 0.0, 2.0 ** -61, 64),
    (150, 1.0, 2.0 ** 61, 64), (2000, 8.0, 2.0 ** -10, 64)])
def test_merges(n, box, r2, capacity):
    ref = same(W.collide_inputs(n, seed=n + 5, box=box), dict(dt=0.01, eps2=0.01, r2_merge=r2), 4, capacity)
    if n >= 200 and r2 > 2.0 ** -60:
        assert ref.merges > 0


@pytest.mark.parametrize("flags", [C.DO_PERSISTENT, C.DO_PLAIN, C.DO_PERSISTENT | C.GRAPH])
def test_merges_with_a_crowd(flags):
    # 40 bodies at one point among spread ones: some wavefronts' lanes walk, some scan.
    inp = W.collide_inputs(700, seed=8, box=2.0)
    inp.x[100:700:15], inp.y[100:700:15] = 0.5, 0.75
    ref = same(inp, W.COLLIDE_PARAMS, 12, flags=flags)
    assert ref.merges >= 39


def test_merges_in_the_least_buffer():
    assert same(W.collide_inputs(500, seed=3, box=0.4), W.COLLIDE_PARAMS, 4, least=True).merges > 0


@pytest.mark.parametrize("x,y", [(1.0e9, 0.0), (0.0, -3.0e38), (np.inf, 1.0), (0.5, np.nan), (2.0 ** 20 / 75, 0.0)])
def test_merges_with_a_far_body(x, y):
    inp = W.collide_inputs(400, seed=4, box=0.5)
    inp.x[77], inp.y[77] = x, y
    assert same(inp, W.COLLIDE_PARAMS, 3).merges > 0 or not np.isfinite(x + y)


def test_merges_across_negative_cells():
    inp = W.collide_inputs(600, seed=6, box=0.4)
    inp.x -= np.float32(0.2)
    inp.y -= np.float32(0.2)
    assert same(inp, W.COLLIDE_PARAMS, 5).merges > 0
