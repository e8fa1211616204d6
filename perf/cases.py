"""Workloads whose speed is followed: what users of this package have it do.

Every case goes through the package's public entry points (`Solver`,
`Group`), from a window of ten sweeps on a grid of ten thousand cells to a
refinement step on 2^30 cells.  Five kinds of use:

  window   fields stay loaded; `sweeps` iterations, the iterate read back
  steps    the same as single calls: pack, exchange, unpack, sweep
  solve    load, solve (fixed count with a residual history, or to a
           relative tolerance), read back
  refine   load, mixed-precision refinement, read back
  group    many grids in shared launches: residual checks and windows,
           every member's iterate read back

`listed()` gives the named cases, `draw(rng)` others of the same ranges.
Inputs: Dirichlet values uniform in [0, 1), a source uniform in [-1, 1); the
first iterate is zero inside (a new solve) or uniform in [0, 1) (a restart).
"""
from __future__ import annotations

import math
import random

import torch

from paper_2102_12416_amd import Group, Solver

DEVICE = "cuda:0"


# ------------------------------------------------------------------ the cases

def _case(name, kind, nx, ny, nz, **kw):
    c = dict(kind=kind, nx=nx, ny=ny, nz=nz, bx=0, by=0, bz=0, cuts=0, mode="fused", source=False, depth=1,
             storage="f64", sweeps=10, warm=True)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # A handful of sweeps and a residual on a grid of a few thousand
        # cells, as a smoother or an inner step of a larger program calls
        # it: launches and latency are all there is.
        _case("window_31x24x17", "window", 31, 24, 17, sweeps=10, residual=True),
        # The package's smallest benchmark: 64^3, one block, default
        # options, 100 iterations with a residual every 10.
        _case("solve_64_history", "solve", 64, 64, 64, mode="staged", sweeps=100, check=10, warm=False),
        # A small solve to a tolerance, three sweeps per launch, ragged
        # edges, with a source: the served requests of the lower end.
        _case("solve_tol_48x33x29", "solve", 48, 33, 29, source=True, depth=3, sweeps=5000, check=50, rtol=1e-6,
              warm=False),
        # The benchmark grid: 512^3 in 2 x 2 x 2 blocks, one launch per
        # iteration, in the benchmark's tile.
        _case("fused_512_2x2x2", "window", 512, 512, 512, bx=256, by=256, bz=256, sweeps=30, tx=256, ty=8, tz=256),
        # An uneven rectilinear decomposition (block edges 32 to 160) in the
        # default tile.
        _case("fused_uneven_420x401x390", "window", 420, 401, 390, cuts=5, sweeps=20),
        # The staged calls one by one, as a program that moves its own halos
        # does, over ragged blocks of 64 cells, and a residual at the end.
        _case("staged_steps_300x260x281", "steps", 300, 260, 281, bx=64, by=64, bz=64, mode="staged", sweeps=10,
              residual=True),
        # One GPU's share of the paper's weak-scaling base as one block,
        # three sweeps per launch, default shape.
        _case("share_3_per_launch", "window", 512, 768, 1536, depth=3, sweeps=12),
        # A mid-size ragged block with a source, two sweeps per launch.
        _case("window_2_per_launch_385x250x333", "window", 385, 250, 333, source=True, depth=2, sweeps=20),
        # Binary32 refinement of a mid-size grid, one sweep per launch.
        _case("refine_f32_384x320x448", "refine", 384, 320, 448, source=True, storage="f32", sweeps=100, inner=50),
        # One outer step of bfloat16 refinement at 1024^3, three inner sweeps
        # per launch: the largest grid of the benchmark.
        _case("refine_bf16_1024", "refine", 1024, 1024, 1024, source=True, storage="bf16", depth=3, sweeps=50,
              inner=50),
        # 256 small grids with a source, each kept on one compute unit:
        # windows of 500 sweeps with a check between them.
        _case("group_resident_256x32", "group", 32, 32, 32, source=True, members=256, resident=True, sweeps=2000,
              check=500),
        # A serving lane: 48 grids of edges 32 to 96, half of them refined in
        # binary32, three sweeps per launch, a check every 50 sweeps.
        _case("group_serving_48", "group", 96, 96, 96, source=True, depth=3, members=48, refined=True, sweeps=100,
              check=50),
    ]


def _edge(rng, lo, hi):
    """A size spread over the logarithm of [lo, hi]; most are odd or ragged."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["window", "window", "blocks", "blocks", "steps", "solve", "solve", "refine", "refine", "group",
                       "group"])
    if kind == "window":
        # one block, any number of sweeps per launch
        n = [_edge(rng, 16, 640) for _ in range(3)]
        return _case("", "window", *n, source=rng.random() < 0.5, depth=rng.choice([1, 2, 3, 3]),
                     sweeps=rng.randint(6, 40), residual=rng.random() < 0.5)
    if kind == "blocks":
        # decomposed, fused: equal blocks (the last of an axis ragged) or
        # rectilinear cuts
        n = [_edge(rng, 96, 560) for _ in range(3)]
        if rng.random() < 0.5:
            return _case("", "window", *n, cuts=rng.randint(1, 10 ** 6), source=rng.random() < 0.3,
                         sweeps=rng.randint(6, 30))
        b = [min(v, _edge(rng, 40, 256)) for v in n]
        return _case("", "window", *n, bx=b[0], by=b[1], bz=b[2], source=rng.random() < 0.3,
                     sweeps=rng.randint(6, 30))
    if kind == "steps":
        n = [_edge(rng, 48, 400) for _ in range(3)]
        b = [min(v, _edge(rng, 32, 200)) for v in n]
        return _case("", "steps", *n, bx=b[0], by=b[1], bz=b[2], mode="staged", source=rng.random() < 0.3,
                     sweeps=rng.randint(3, 12), residual=True)
    if kind == "solve":
        n = [_edge(rng, 12, 110) for _ in range(3)]
        depth = rng.choice([1, 2, 3, 3])
        if rng.random() < 0.5:
            return _case("", "solve", *n, source=rng.random() < 0.5, depth=depth, sweeps=rng.randint(40, 200),
                         check=rng.choice([10, 20, 25]), warm=False)
        return _case("", "solve", *n, source=True, depth=depth, sweeps=2000, check=50, rtol=10 ** rng.uniform(-5, -3),
                     warm=False)
    if kind == "refine":
        n = [_edge(rng, 32, 512) for _ in range(3)]
        return _case("", "refine", *n, source=True, storage=rng.choice(["f64", "f32", "f32", "bf16", "bf16"]),
                     depth=rng.choice([1, 2, 3]), sweeps=rng.choice([50, 100]), inner=50)
    if rng.random() < 0.5:
        e = _edge(rng, 8, 32)
        return _case("", "group", e, e, e, source=rng.random() < 0.5, members=rng.randint(32, 320), resident=True,
                     sweeps=1000, check=rng.choice([100, 250, 500]))
    e = _edge(rng, 32, 128)
    return _case("", "group", e, e, e, source=True, depth=rng.choice([1, 2, 3]), members=rng.randint(4, 56),
                 refined=rng.random() < 0.5, sweeps=100, check=50)


# ------------------------------------------------------------------ inputs

def _cuts(case):
    """Block edges of 32 to 160 cells along each axis."""
    rng = random.Random(case["cuts"])
    out = []
    for n in (case["nx"], case["ny"], case["nz"]):
        left, cut = n, []
        while left > 160:
            e = min(_edge(rng, 32, 160), left - 32)
            cut.append(e)
            left -= e
        out.append(cut + [left])
    return out


def _fields(grid, seed, source, warm):
    """First iterate (padded) and source (padded, its shell unused) of one grid."""
    nx, ny, nz = grid
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(int(seed))
    u = torch.rand((nz + 2, ny + 2, nx + 2), dtype=torch.float64, device=DEVICE, generator=gen)
    if not warm:
        u[1:-1, 1:-1, 1:-1] = 0.0
    b = None
    if source:
        b = torch.rand((nz + 2, ny + 2, nx + 2), dtype=torch.float64, device=DEVICE, generator=gen)
        b.mul_(2.0).sub_(1.0)
    return u, b


def _members(case):
    """Grid and refinement storage of every member of a group: a quarter
    each at the full, three quarters, two thirds and half the edge, the
    third ragged; every second one refined where the case says so."""
    e = case["nx"]
    sizes = [(e, e, e), (3 * e // 4,) * 3, (max(1, 2 * e // 3), max(1, 2 * e // 3 - 1), max(1, 2 * e // 3 + 1)),
             (max(1, e // 2),) * 3]
    return [(sizes[i % 4], bool(case.get("refined")) and (i // 4) % 2 == 1) for i in range(case["members"])]


def _solver(case, grid, stream=None, refined=None):
    kw = dict(mode=case["mode"], with_source=case["source"], stream=stream)
    if case["depth"] > 1 and refined is None:
        kw["temporal"] = 3 if case["depth"] == 3 else True
    if case["kind"] == "refine":
        kw["ir_dtype"] = case["storage"]
    if refined:
        kw["ir_dtype"] = "f32"
    if case["cuts"]:
        kw["cuts"] = _cuts(case)
    elif case["bx"]:
        kw["block_dims"] = (case["bx"], case["by"], case["bz"])
    return Solver(grid, **kw)


def prepare(case, seed):
    if case["kind"] == "group":
        stream = torch.cuda.Stream(device=DEVICE)
        solvers = []
        for i, (grid, refined) in enumerate(_members(case)):
            s = _solver(case, grid, stream=stream, refined=refined)
            s.load(*_fields(grid, seed * 1000 + i, case["source"], case["warm"]))
            solvers.append(s)
        group = Group(solvers, stream=stream, resident=bool(case.get("resident")),
                      temporal={1: False, 2: True, 3: 3}[case["depth"]])
        return dict(case=case, solvers=solvers, group=group)
    grid = (case["nx"], case["ny"], case["nz"])
    u, b = _fields(grid, seed, case["source"], case["warm"])
    s = _solver(case, grid)
    if case.get("tx"):
        s.set_tiles(case["tx"], case["ty"], case["tz"])
    if case["kind"] in ("window", "steps"):
        s.load(u, b)
        return dict(case=case, solver=s)
    return dict(case=case, solver=s, u=u, b=b)


# ------------------------------------------------------------------ one pass

def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "group":
        group = state["group"]
        for _ in range(case["sweeps"] // case["check"]):
            group.check(1e-12, 10 ** 9)
            group.iterate(case["check"])
        if case.get("refined"):
            group.check(1e-12, 10 ** 9)         # the refined members' last update
        fields = [s.store().reshape(-1) for s in state["solvers"]]
        return torch.cat(fields)
    s = state["solver"]
    out = {}
    if kind == "window":
        s.iterate(case["sweeps"])
    elif kind == "steps":
        for _ in range(case["sweeps"]):
            s.pack_faces()
            s.exchange()
            s.unpack_faces()
            s.sweep()
    elif kind == "solve":
        s.load(state["u"], state["b"])
        rtol = case.get("rtol", 0.0)
        info = s.solve(rtol=rtol, max_iter=case["sweeps"], check_every=case["check"], history=rtol == 0.0)
        out["iters"] = int(info["iters"])
        if rtol == 0.0:
            out["history"] = torch.tensor(info["history"], dtype=torch.float64)
    else:
        s.load(state["u"], state["b"])
        info = s.solve_ir(inner=case["inner"], rtol=0.0, max_inner=case["sweeps"])
        out["iters"] = int(info["iters"])
    if case.get("residual"):
        out["residual"] = s.residual()
    out["u"] = s.store()
    return out


# ------------------------------------------------------------------ what it cannot do without

def work(case):
    if case["kind"] == "group":
        cells = sum(g[0] * g[1] * g[2] for g, _ in _members(case))
    else:
        cells = case["nx"] * case["ny"] * case["nz"]
    sweeps = case["sweeps"]
    if "rtol" in case:
        # sweeps to the tolerance, from the spectral radius of the sweep
        rho = sum(math.cos(math.pi / (case[a] + 1)) for a in ("nx", "ny", "nz")) / 3
        sweeps = min(sweeps, math.ceil(math.log(case["rtol"]) / math.log(rho)))
    arrays = 2 + (1 if case["source"] else 0)     # first iterate and source in, iterate out
    return {"bytes": 8.0 * arrays * cells, "flops": float(6 + (1 if case["source"] else 0)) * cells * sweeps}


# ------------------------------------------------------------------ the same in plain torch, 64 bits

def _neighbours(u):
    s = u[..., 1:-1, 1:-1, :-2] + u[..., 1:-1, 1:-1, 2:]
    s += u[..., 1:-1, :-2, 1:-1]
    s += u[..., 1:-1, 2:, 1:-1]
    s += u[..., :-2, 1:-1, 1:-1]
    s += u[..., 2:, 1:-1, 1:-1]
    return s


def _inside(u):
    return u[..., 1:-1, 1:-1, 1:-1]


def _sweep(u, b):
    s = _neighbours(u)
    if b is not None:
        s += _inside(b)
    _inside(u).copy_(s / 6.0)


def _residual(u, b):
    s = _neighbours(u)
    if b is not None:
        s = _inside(b) + s
    return float((s - 6.0 * _inside(u)).square().sum().sqrt())


def exact(case, seed):
    if case["kind"] == "group":
        members = _members(case)
        fields = [_fields(g, seed * 1000 + i, case["source"], case["warm"]) for i, (g, _) in enumerate(members)]
        out = [None] * len(members)
        for grid in {g for g, _ in members}:      # the members of one size together
            at = [i for i, (g, _) in enumerate(members) if g == grid]
            u = torch.stack([fields[i][0] for i in at])
            b = torch.stack([fields[i][1] for i in at]) if case["source"] else None
            for _ in range(case["sweeps"]):
                _sweep(u, b)
            for k, i in enumerate(at):
                out[i] = u[k].reshape(-1)
        return torch.cat(out)
    u, b = _fields((case["nx"], case["ny"], case["nz"]), seed, case["source"], case["warm"])
    out = {}
    done = 0
    if case["kind"] == "solve":
        rtol, check = case.get("rtol", 0.0), case["check"]
        history, first = [], None
        while done <= case["sweeps"]:
            if done % check == 0 or done == case["sweeps"]:
                r = _residual(u, b)
                history.append(r)
                first = r if first is None else first
                if rtol > 0.0 and r <= rtol * first:
                    break
            if done == case["sweeps"]:
                break
            _sweep(u, b)
            done += 1
        if rtol == 0.0:
            out["history"] = torch.tensor(history, dtype=torch.float64)
    else:
        for done in range(1, case["sweeps"] + 1):
            _sweep(u, b)
    if case["kind"] in ("solve", "refine"):
        out["iters"] = done
    if case.get("residual"):
        out["residual"] = _residual(u, b)
    out["u"] = u
    return out
