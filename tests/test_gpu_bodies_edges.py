"""Force do-all at the edges of its tiles and of its arithmetic's two forms,
against the oracle: every operation is rounded once in the oracle's order, so
the results are equal bit for bit (NaN wherever the oracle has NaN)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
from paper_1809_07444_amd import _capi as C  # noqa: E402
from paper_1809_07444_amd import apps  # noqa: E402
from synth import workloads as W  # noqa: E402

FIELDS = ("x", "y", "vx", "vy", "m")


def same(inp, params, steps, capacity=64, flags=C.DO_PERSISTENT):
    sim = apps.Collisions(inp, params, capacity=capacity)
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
