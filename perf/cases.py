"""Timed cases of the framework: what a program built on it runs, over the range of
sizes it meets.  Every case resets its heap, creates the initial objects, runs the
application's steps and hands the canonical state back in device memory, as bench.py
and the tests drive the same entry points; the inputs come from the seed alone."""
from __future__ import annotations

import functools
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_1809_07444_amd import _capi as C
from paper_1809_07444_amd import apps, batch, heap, serve

# Rule constants of the applications, as the framework's own benchmark runs them.
SUGAR = dict(max_age=100, repro_min=20, fertile_min=10, fertile_max=60)
TRAFFIC = dict(vmax=5, p_slow24=1 << 22, p_in24=1 << 23)
COLLIDE = dict(dt=0.01, eps2=0.01, r2_merge=0.0001)
NBODY = dict(dt=0.01, eps2=0.01, r2_merge=0.0)
WATOR = dict(fish_breed=3, shark_breed=10, starve=3)


def listed():
    return [
        # The alloc / do-all microbenchmark at its standard size: every kernel is short,
        # so launches and the latency of the allocation path count.
        dict(name="micro_64k", kind="micro", n=65536, blocks=4096, steps=10),
        # The same step on a heap far larger than the caches: the bandwidth case.
        dict(name="micro_64m", kind="micro", n=1 << 26, blocks=1 << 22, steps=2),
        # Host-driven use of the heap: bulk new, field access, a deleting do-all, new
        # into the holes, bulk delete, gather.
        dict(name="heap_1m", kind="heap", n=1000003),
        # The smallest simulation: one 64 x 64 world, launched eagerly (the default).
        dict(name="gol_64", kind="gol", side=64, steps=20, graph=False, capacity=64),
        # One ordinary world, replayed from graphs.
        dict(name="gol_1024", kind="gol", side=1024, steps=200, graph=True, capacity=64),
        # 256 uneven worlds in one heap: the benchmark's default workload.
        dict(name="gol_batch_256", kind="batch", worlds=256, lo=64, hi=1024, steps=100),
        # Agents with births and deaths on a large grid.
        dict(name="sugarscape_2048", kind="sugar", side=2048, agents=1 << 20, steps=100),
        # Many roads: short kernels, a few objects created and deleted per step.
        dict(name="traffic_1024", kind="traffic", roads=1024, length=1024, steps=100),
        # A few thousand merging bodies: far fewer wavefronts than the chip holds.
        dict(name="collisions_4096", kind="bodies", n=4096, merge=True, spread=1.0, steps=50),
        # Bodies without merging at the benchmark's size: arithmetic bound.
        dict(name="nbody_65536", kind="bodies", n=65536, merge=False, spread=1.0, steps=5),
        # Two object types with births, meals and starvation.
        dict(name="wator_2048", kind="wator", side=2048, steps=50),
        # Continuous batching: episodes of both pools admitted, stepped together, retired.
        dict(name="serve_8", kind="serve", episodes=8, side=384, steps=40),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["micro", "heap", "gol", "batch", "sugar", "traffic", "bodies", "bodies", "wator", "serve"])
    if kind == "micro":
        n = _log(rng, 300, 1 << 24)
        return dict(kind=kind, n=n, blocks=max(64, n // 16 + rng.randrange(64)), steps=rng.randint(2, 10))
    if kind == "heap":
        return dict(kind=kind, n=_log(rng, 1000, 1 << 22))
    if kind == "gol":
        return dict(kind=kind, side=_log(rng, 16, 1500), steps=rng.randint(5, 60), graph=rng.random() < 0.75,
                    capacity=rng.choice([64, 64, 64, 32]))
    if kind == "batch":
        return dict(kind=kind, worlds=_log(rng, 2, 200), lo=rng.randint(16, 64), hi=rng.randint(128, 900),
                    steps=rng.randint(5, 40))
    if kind == "sugar":
        side = _log(rng, 64, 2048)
        return dict(kind=kind, side=side, agents=int(side * side * rng.uniform(0.05, 0.3)), steps=rng.randint(5, 60))
    if kind == "traffic":
        return dict(kind=kind, roads=_log(rng, 8, 2048), length=_log(rng, 64, 2048), steps=rng.randint(10, 100))
    if kind == "bodies":
        n = _log(rng, 100, 40000)
        return dict(kind=kind, n=n, merge=rng.random() < 0.6, spread=round(rng.uniform(0.3, 1.0), 3),
                    steps=rng.randint(2, 10))
    if kind == "wator":
        return dict(kind=kind, side=_log(rng, 64, 2048), steps=rng.randint(5, 40))
    return dict(kind=kind, episodes=rng.randint(2, 8), side=_log(rng, 64, 512), steps=rng.randint(10, 40))


@functools.lru_cache(maxsize=None)
def _stream():
    """The program's one work stream: its simulations run one after the other."""
    return torch.cuda.Stream()


# ------------------------------------------------------------------ inputs --

def _gen(seed, salt=0):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + salt) & 0x7FFFFFFFFFFFFFFF)
    return g


def _u(g, *shape):
    return torch.rand(shape, generator=g, device="cuda")


def _int(g, lo, hi, *shape):
    return torch.randint(lo, hi + 1, shape, generator=g, device="cuda", dtype=torch.int32)


def _np(t):
    return t.cpu().numpy()


def _micro_inputs(case, seed):
    g = _gen(seed, 1)
    n, steps = case["n"], case["steps"]
    r = (n + 2) // 3
    return dict(x0=_u(g, n), v0=torch.randn(n, generator=g, device="cuda"), xs=_u(g, steps, r),
                vs=torch.randn((steps, r), generator=g, device="cuda"))


def _heap_inputs(case, seed):
    g = _gen(seed, 2)
    n = case["n"]
    return _u(g, n), _u(g, (n + 2) // 3)


def _grid(side, seed, salt):
    return (_u(_gen(seed, salt), side, side) < 0.1).to(torch.uint8)


def _sides(case):
    """Uneven sides, log-uniform between lo and hi (a golden-ratio sequence: the same
    for every seed)."""
    lo, hi = case["lo"], case["hi"]
    return [int(round(lo * (hi / lo) ** ((0.5 + 0.6180339887498949 * i) % 1.0))) for i in range(case["worlds"])]


def _batch_grids(case, seed):
    sides = _sides(case)
    flat = (_u(_gen(seed, 4), sum(s * s for s in sides)) < 0.1).to(torch.uint8)
    return [p.view(s, s) for p, s in zip(torch.split(flat, [s * s for s in sides]), sides)]


def _sugar_inputs(side, agents, seed, salt=5):
    g = _gen(seed, salt)
    n = side * side
    cap = _int(g, 0, 4, n)
    occ = torch.zeros(n, dtype=torch.uint8, device="cuda")
    occ[torch.randperm(n, generator=g, device="cuda")[:agents]] = 1
    m = occ.to(torch.int32)
    traits = [_int(g, lo, hi, n) * m for lo, hi in ((5, 25), (1, 4), (1, 6), (0, SUGAR["max_age"] - 1))]
    cap, occ = _np(cap), _np(occ)
    return SimpleNamespace(side=side, n_agents=agents, seed=int(seed) & 0xFFFFFFFF, sugar=cap.copy(), cap=cap, occ=occ,
                           **dict(zip(("a_sugar", "a_metab", "a_vision", "a_age"), map(_np, traits))))


def _bodies(case, seed):
    """Bodies uniform in a square (a quarter of a thousandth mass each on average); a
    spread below 1 packs them more densely, so that more of them merge."""
    g = _gen(seed, 6)
    n = case["n"]
    box = 16.0 * math.sqrt(n / 16384.0) * case["spread"]
    xy = [_u(g, n) * box for _ in range(2)]
    v = [_u(g, n) - 0.5 for _ in range(2)]
    m = _int(g, 1, 4, n).to(torch.float32) / 1024
    return SimpleNamespace(n=n, **dict(zip(("x", "y", "vx", "vy", "m"), map(_np, xy + v + [m]))))


def _episodes(case, seed):
    """Seven Game-of-Life worlds in ten, the others Sugarscape, sides around the case's."""
    specs, inputs = [], {}
    for i in range(case["episodes"]):
        kind = "sugar" if i % 3 == 2 else "gol"
        side = max(16, int(case["side"] * (0.5 + 0.75 * ((0.3 + 0.618 * i) % 1.0))))
        length = max(2, case["steps"] - (i * 7) % (case["steps"] // 2 + 1))
        specs.append(SimpleNamespace(eid=i, kind=kind, side=side, length=length, seed=int(seed) * 64 + i,
                                     agents=side * side // 5, arrival=0.0))
        inputs[i] = (_np(_grid(side, seed, 100 + i)) if kind == "gol"
                     else _sugar_inputs(side, side * side // 5, seed, 100 + i))
    return specs, inputs


# ----------------------------------------------------------------- prepare --

def prepare(case, seed):
    kind = case["kind"]
    flags = C.DO_PERSISTENT | (C.GRAPH if case.get("graph", True) else 0)
    s = SimpleNamespace(kind=kind, case=case, flags=flags)
    if kind == "micro":
        t = _micro_inputs(case, seed)
        s.inp = SimpleNamespace(n_init=case["n"], steps=case["steps"], n_renew=t["xs"].shape[1],
                                **{k: _np(v) for k, v in t.items()})
        s.sim = apps.MicroBench(s.inp, num_blocks=case["blocks"])
    elif kind == "heap":
        n = case["n"]
        s.vals, s.again = _heap_inputs(case, seed)
        s.heap = heap.Heap(n // 48 + 256, 64, types=((4, 4),))  # a third more than full blocks need
        s.keys = torch.arange(n, dtype=torch.int32, device="cuda")
        s.gone = torch.arange(1, n, 3, device="cuda")  # handles freed one by one by the caller
    elif kind == "gol":
        s.sim = apps.GameOfLife([_np(_grid(case["side"], seed, 3))], capacity=case["capacity"],
                                stream=_stream())
    elif kind == "batch":
        s.runner = batch.BatchedGol([_np(g) for g in _batch_grids(case, seed)], batch.TuneConfig(wgs_per_cu=16))
        s.sim = s.runner.gol
    elif kind == "sugar":
        s.sim = apps.Sugarscape(_sugar_inputs(case["side"], case["agents"], seed), SUGAR, stream=_stream())
    elif kind == "traffic":
        g = _gen(seed, 7)
        shape = (case["roads"], case["length"])
        vel = torch.where(_u(g, *shape) < 0.15, _int(g, 0, TRAFFIC["vmax"], *shape), -1)
        s.sim = apps.Traffic(SimpleNamespace(roads=case["roads"], length=case["length"], seed=int(seed), vel=_np(vel)),
                             TRAFFIC, stream=_stream())
    elif kind == "bodies":
        s.sim = apps.Collisions(_bodies(case, seed), COLLIDE if case["merge"] else NBODY,
                              stream=_stream())
    elif kind == "wator":
        g = _gen(seed, 8)
        side = case["side"]
        u = _u(g, side, side)
        k = torch.where(u < 0.3, 1, torch.where(u < 0.35, 2, 0)).to(torch.int32)
        age = torch.where(k == 1, _int(g, 0, WATOR["fish_breed"] - 1, side, side),
                          torch.where(k == 2, _int(g, 0, WATOR["shark_breed"] - 1, side, side), 0))
        energy = torch.where(k == 2, _int(g, 1, WATOR["starve"], side, side), 0)
        s.sim = apps.Wator(SimpleNamespace(side=side, seed=int(seed), kind=_np(k), age=_np(age), energy=_np(energy)),
                           WATOR, stream=_stream())
    else:
        s.specs, s.inputs = _episodes(case, seed)
        s.server = serve.Server(rules=SUGAR)
    torch.cuda.synchronize()
    return s


# --------------------------------------------------------------------- run --

def run(s):
    if s.kind == "micro":
        s.sim.run()
        n, h = s.inp.n_init, s.sim.heap
        (x, px), (v, _) = h.gather(0, 0, 1, n), h.gather(0, 0, 2, n)
        return [x.view(torch.float32), v.view(torch.float32), px]
    if s.kind == "heap":
        h, n = s.heap, s.case["n"]
        h.reset()
        objs = h.alloc_n(0, n)
        h.field_write(0, 0, objs, s.keys)
        h.field_write(0, 1, objs, s.vals)
        h.delete_if_mod(0, 0, 3, 0)
        more = h.alloc_n(0, s.again.numel())
        h.field_write(0, 0, more, s.keys[::3])
        h.field_write(0, 1, more, s.again)
        kept = h.field_read(0, 1, objs[s.gone])
        h.free_n(objs[s.gone])
        out, present = h.gather(0, 0, 1, n)
        return [out.view(torch.float32), present, kept.view(torch.float32)]
    if s.kind == "serve":
        _, results, _ = s.server.run(s.specs, lambda e: s.inputs[e.eid])
        return [results[e.eid] for e in s.specs]
    sim, steps = s.sim, s.case["steps"]
    st = sim.heap._s()
    if s.kind in ("gol", "batch"):
        if s.kind == "batch":
            s.runner.run(steps)
        else:
            sim.init()
            sim.step(steps, s.flags)
        C.check(sim.lib.dsoar_gol_read(sim.g, sim.out.data_ptr(), st), "dsoar_gol_read")
        return sim.out
    sim.init()
    sim.step(steps, s.flags)
    if s.kind == "sugar":
        C.check(sim.lib.dsoar_sugar_read(sim.s, *[t.data_ptr() for t in sim.out], None, st), "dsoar_sugar_read")
    elif s.kind == "traffic":
        C.check(sim.lib.dsoar_traffic_read(sim.t, sim.out.data_ptr(), st), "dsoar_traffic_read")
    elif s.kind == "bodies":
        C.check(sim.lib.dsoar_collide_read(sim.c, *[t.data_ptr() for t in sim.out], st), "dsoar_collide_read")
    else:
        C.check(sim.lib.dsoar_wator_read(sim.w, *[t.data_ptr() for t in sim.out], st), "dsoar_wator_read")
    return sim.out


# -------------------------------------------------------------------- work --

def work(case):
    """Inputs read once, results written once, and per step the state that the step's
    rules read and write, each once: live objects' fields, grid cells (a Game-of-Life
    cell is one bit)."""
    kind, steps = case["kind"], case.get("steps", 1)
    if kind == "micro":  # per step: update x, cull by id, create a third again
        n = case["n"]
        return {"bytes": n * 20 + steps * (n * 16 + n / 3 * 20) + n * 18, "flops": 2.0 * n * steps}
    if kind == "heap":
        n = case["n"]
        return {"bytes": n * (8 + 8 + 4 + 16 / 3 + 4 + 13), "flops": 0}
    if kind in ("gol", "batch"):
        cells = sum(x * x for x in (_sides(case) if kind == "batch" else [case["side"]]))
        return {"bytes": cells * (2 + steps * 0.25), "flops": 0}
    if kind == "sugar":
        cells = case["side"] ** 2
        return {"bytes": cells * (25 + 21 + steps * 3) + case["agents"] * 28 * (1 + steps * 2), "flops": 0}
    if kind == "traffic":
        cells = case["roads"] * case["length"]
        return {"bytes": cells * 8 + cells * 0.15 * 16 * (1 + steps), "flops": 0}
    if kind == "bodies":
        n = float(case["n"])
        return {"bytes": n * 20 * 2 + n * 64 * steps, "flops": 13 * n * n * steps}
    if kind == "wator":
        cells = case["side"] ** 2
        return {"bytes": cells * (24 + steps * 2) + cells * 0.35 * 16 * (1 + 2 * steps), "flops": 0}
    cells = sum(float(e) for e in [case["side"] ** 2] * case["episodes"])
    return {"bytes": cells * (10 + 2 * steps), "flops": 0}


# ------------------------------------------------------------------- exact --

def _life(grid, gens):
    for _ in range(gens):
        n = sum(torch.roll(grid, (dy, dx), (0, 1)) for dy in (-1, 0, 1) for dx in (-1, 0, 1) if dy or dx)
        grid = ((n == 3) | ((n == 2) & (grid == 1))).to(torch.uint8)
    return grid.reshape(-1)


def _bodies64(case, seed):
    """The bodies' rules in 64 bits: forces from every body of positive mass, then the
    moves; a body with no live body of lower id in the merge radius is a root, the
    others merge into the lowest root in theirs."""
    b = _bodies(case, seed)
    x, y, vx, vy, m = (torch.from_numpy(getattr(b, k)).cuda().double() for k in ("x", "y", "vx", "vy", "m"))
    # The parameters are 32-bit values of the interface.
    dt, eps2, r2 = (float(np.float32((COLLIDE if case["merge"] else NBODY)[k])) for k in ("dt", "eps2", "r2_merge"))
    n, ids = b.n, torch.arange(b.n, device="cuda")
    rows = max(1, (1 << 27) // n)
    for _ in range(case["steps"]):
        ax, ay = torch.zeros_like(x), torch.zeros_like(y)
        for i in range(0, n, rows):
            dx, dy = x[None, :] - x[i:i + rows, None], y[None, :] - y[i:i + rows, None]
            d = dx * dx + dy * dy + eps2
            f = m[None, :] / (d * d.sqrt())
            ax[i:i + rows], ay[i:i + rows] = (f * dx).sum(1), (f * dy).sum(1)
        live = m > 0
        vx, vy = torch.where(live, vx + dt * ax, vx), torch.where(live, vy + dt * ay, vy)
        x, y = torch.where(live, x + dt * vx, x), torch.where(live, y + dt * vy, y)
        if r2 <= 0:
            continue
        pairs = []
        for i in range(0, n, rows):
            dx, dy = x[None, :] - x[i:i + rows, None], y[None, :] - y[i:i + rows, None]
            near = (dx * dx + dy * dy < r2) & live[None, :] & live[i:i + rows, None]
            p = near.nonzero()
            pairs.append(torch.stack([p[:, 0] + i, p[:, 1]], 1))
        p = torch.cat(pairs)
        p = p[p[:, 0] != p[:, 1]]
        root = live.clone()
        root[p[p[:, 1] < p[:, 0]][:, 0]] = False
        q = p[~root[p[:, 0]] & root[p[:, 1]]]
        into = torch.full((n,), n, device="cuda").scatter_reduce_(0, q[:, 0], q[:, 1], "amin")
        gone = (into < n) & live
        src, dst = ids[gone], into[gone]
        if not src.numel():
            continue
        M = m.clone().index_add_(0, dst, m[src])
        sums = [(m * u).index_add_(0, dst, (m * u)[src]) / M for u in (x, y, vx, vy)]
        took = torch.zeros_like(live)
        took[dst] = True
        x, y, vx, vy = (torch.where(took, a, u) for a, u in zip(sums, (x, y, vx, vy)))
        m = torch.where(took, M, m)
        m[gone] = 0
    return [x, y, vx, vy, m]


def exact(case, seed):
    kind = case["kind"]
    if kind == "micro":
        t = {k: v.double() for k, v in _micro_inputs(case, seed).items()}
        x, v, dt = t["x0"], t["v0"], float(np.float32(0.01))  # the step's 32-bit constant
        for k in range(case["steps"]):
            x = x + dt * v
            x[::3], v[::3] = t["xs"][k], t["vs"][k]
        return [x, v, torch.ones(case["n"], dtype=torch.uint8)]
    if kind == "heap":
        n = case["n"]
        vals, again = _heap_inputs(case, seed)
        out, present = vals.clone(), torch.ones(n, dtype=torch.uint8, device="cuda")
        out[::3] = again
        kept = vals[1::3].clone()
        out[1::3], present[1::3] = 0, 0
        return [out.double(), present, kept.double()]
    if kind == "gol":
        return _life(_grid(case["side"], seed, 3), case["steps"])
    if kind == "batch":
        return torch.cat([_life(g, case["steps"]) for g in _batch_grids(case, seed)])
    if kind == "bodies":
        return _bodies64(case, seed)
    return None  # whole numbers under rules with draws of their own: they are compared as they are
