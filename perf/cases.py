"""What is timed: solves as programs run them, through the public entry points.

Each case is one kind of call over sizes, decompositions and options that the
solver, the batch, the pool and the allocation-free entry point are used with:

  solve    a Solver kept by the program: load an interior that is resident on
           the device, run, read the interior back to the device.  `check` > 0
           reads the residual every `check` sweeps (an iteration to tolerance),
           0 only after the last one.
  serial   one request from scratch, as a queue of plain solves handles it:
           create the solver, run, copy the result to the host, close.
  batch    independent problems of uneven sizes, advanced together.
  pool     requests of different sizes served by continuous batching, results
           in page-locked host memory.
  noalloc  the one-shot solve on memory that the caller owns.

Grid axes are x, y, z with x fastest; dense arrays have shape (nz, ny, nx).
"""
import math
import random

import numpy as np
import torch

from paper_2202_11819_amd import api, j3d
from paper_2202_11819_amd import workloads as W

DEV = "cuda"


def _solve(name, n, nblk=(1, 1, 1), iters=50, mode="graph", check=0, uneven=0, bc=False,
           faces=False):
    case = {"kind": "solve", "nx": n[0], "ny": n[1], "nz": n[2], "bx": nblk[0], "by": nblk[1], "bz": nblk[2],
            "iters": iters, "mode": mode, "check": check, "uneven": uneven, "bc": bc, "faces": faces}
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # a small iteration to tolerance: every 50 sweeps the program looks at
        # the residual; launches and the host round trip are what it waits for
        _solve("tiny_checked", (33, 35, 31), iters=200, check=50, bc=True),
        # the small plain run: one block, zero boundary, 100 sweeps
        _solve("small_64", (64, 64, 64), iters=100),
        # one block with a boundary given cell by cell, an odd non-cubic grid
        _solve("faces_odd", (157, 211, 183), iters=120, faces=True),
        # the over-decomposed benchmark grid in the default mode
        _solve("odf_512", (512, 512, 512), (8, 8, 8), iters=100),
        # kernel fusion strategy C driven sweep by sweep
        _solve("fused_256", (256, 256, 256), (4, 4, 4), iters=50, mode="fused"),
        # the largest grid, blocks of 128^3
        _solve("grid_1024", (1024, 1024, 1024), (8, 8, 8), iters=30),
        # blocks of uneven extents, 100..160 cells per axis
        _solve("uneven_640", (640, 640, 640), (5, 5, 5), iters=50, uneven=100, bc=True),
        # the undivided grid with several sweeps per launch asked for
        _solve("two_sweep_512", (512, 512, 512), iters=100, mode="two_sweep"),
        # the one-shot solve of a program that may not allocate
        {"name": "noalloc_192", "kind": "noalloc", "nx": 192, "ny": 160, "nz": 176, "bx": 2, "by": 2, "bz": 2,
         "iters": 50},
        # a served request handled alone, result on the host
        {"name": "serial_request", "kind": "serial", "nx": 211, "ny": 173, "nz": 190, "iters": 200},
        # many small problems at once: 32..256 cells per axis, 100..1000 sweeps
        {"name": "batch_48", "kind": "batch", "count": 48, "lo": 32, "hi": 256, "it_lo": 100, "it_hi": 1000,
         "two_sweep": False, "mix": 7},
        # a served mix: 32..384 cells per axis, residual every 50 sweeps
        {"name": "pool_12", "kind": "pool", "count": 12, "lo": 32, "hi": 384, "it_lo": 50, "it_hi": 600,
         "two_sweep": False, "mix": 11},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(["solve"] * 6 + ["serial", "batch", "pool", "noalloc"])
    if kind == "serial":
        return {"kind": kind, "nx": rng.randint(32, 384), "ny": rng.randint(32, 384), "nz": rng.randint(32, 384),
                "iters": rng.randint(50, 400)}
    if kind == "batch":
        return {"kind": kind, "count": _log_int(rng, 4, 48), "lo": 32, "hi": rng.randint(64, 256), "it_lo": 100,
                "it_hi": rng.randint(200, 1000), "two_sweep": rng.random() < 0.4, "mix": rng.randrange(1 << 20)}
    if kind == "pool":
        return {"kind": kind, "count": rng.randint(2, 12), "lo": 32, "hi": rng.randint(64, 384), "it_lo": 50,
                "it_hi": rng.randint(100, 600), "two_sweep": rng.random() < 0.4, "mix": rng.randrange(1 << 20)}
    # the edge first (logarithmic over the whole range), then each axis around it
    edge = _log_int(rng, 24, 720)
    n = [max(16, min(800, int(edge * math.exp(rng.uniform(-0.35, 0.35))))) for _ in range(3)]
    if kind == "noalloc":
        n = [min(v, 320) for v in n]
        nb = [rng.randint(1, max(1, min(4, v // 24))) for v in n]
        n = [v // b * b for v, b in zip(n, nb)]
        return {"kind": kind, "nx": n[0], "ny": n[1], "nz": n[2], "bx": nb[0], "by": nb[1], "bz": nb[2],
                "iters": rng.randint(10, 100)}
    mode = rng.choice(["graph"] * 5 + ["fused"] * 2 + ["two_sweep"] * 2)
    uneven, nb = 0, [1, 1, 1]
    if mode != "two_sweep" and rng.random() < 0.7:
        be = _log_int(rng, 24, 200)                      # block edge
        nb = [max(1, min(16, round(v / be))) for v in n]
        if max(nb) > 1 and rng.random() < 0.4 and min(v // b for v, b in zip(n, nb)) >= 12:
            uneven = max(4, int(min(v // b for v, b in zip(n, nb)) * 0.8))
        else:
            n = [v // b * b for v, b in zip(n, nb)]
    cells = n[0] * n[1] * n[2]
    most = max(10, min(400, int(16e9 / cells)))
    iters = rng.randint(max(5, most // 8), most)
    check = rng.choice([0, 0, 50, 25]) if cells < 2 ** 24 else 0
    return _solve(None, n, nb, iters, mode, check, uneven, bc=rng.random() < 0.5, faces=rng.random() < 0.2)


# ---- inputs ---------------------------------------------------------------------

def _n(case):
    return case["nx"], case["ny"], case["nz"]


def _split(case):
    """Block extents per axis: an even split (None), or pieces of at least
    `uneven` cells with the rest of the axis spread unevenly over them."""
    if not case.get("uneven"):
        return None
    out = []
    for axis, (n, b) in enumerate(zip(_n(case), (case["bx"], case["by"], case["bz"]))):
        rng = random.Random(1000 * case["uneven"] + 10 * n + axis)
        lo = min(case["uneven"], n // b)
        cuts = sorted(rng.randint(0, n - lo * b) for _ in range(b - 1))
        out.append([lo + y - x for x, y in zip([0] + cuts, cuts + [n - lo * b])])
    return out


def _bc(seed, salt=0):
    rng = random.Random(seed * 7919 + salt)
    return tuple(rng.uniform(-1.0, 1.0) for _ in range(6))


def _interior(case, seed):
    nx, ny, nz = _n(case)
    g = torch.Generator(device=DEV).manual_seed(seed)
    return torch.rand((nz, ny, nx), dtype=torch.float64, device=DEV, generator=g)


def _faces(case, seed):
    """Per-cell boundary values, x-, x+, y-, y+, z-, z+."""
    nx, ny, nz = _n(case)
    rng = np.random.default_rng([seed, 17])
    shapes = [(nz, ny), (nz, ny), (nz, nx), (nz, nx), (ny, nx), (ny, nx)]
    return [rng.uniform(-1.0, 1.0, s) for s in shapes]


def _mix(case, seed):
    """Problems of a batch or pool: sizes and sweep counts from `mix`, boundary
    values and seeded interiors from the seed."""
    rng = np.random.default_rng([case["mix"], 3])
    out = []
    for i in range(case["count"]):
        lo, hi = case["lo"], case["hi"]
        if case["kind"] == "batch":
            n = tuple(int(min(hi, math.floor(lo * (hi / lo) ** rng.uniform()))) for _ in range(3))
            bc = _bc(seed, i + 1)
        else:
            n = tuple(int(v) for v in rng.integers(lo, hi + 1, 3))
            bc = (0.0,) * 6
        out.append(W.Spec(n=n, bc=bc, seed=seed, pid=i, iters=int(rng.integers(case["it_lo"], case["it_hi"] + 1))))
    return out


# ---- passes ---------------------------------------------------------------------

def prepare(case, seed):
    kind = case["kind"]
    if kind == "solve":
        bc = _bc(seed) if case["bc"] else (0.0,) * 6
        s = api.Solver(_n(case), nblk=(case["bx"], case["by"], case["bz"]), split=_split(case), bc=bc, seed=seed)
        if case["faces"]:
            for f, v in enumerate(_faces(case, seed)):
                s.set_face(f, v)
        return {"case": case, "solver": s, "u0": _interior(case, seed)}
    if kind == "serial":
        return {"case": case, "seed": seed}
    if kind == "batch":
        specs = _mix(case, seed)
        return {"case": case, "problems": [W.to_problem(s) for s in specs], "iters": [s.iters for s in specs]}
    if kind == "pool":
        specs = _mix(case, seed)
        problems = [W.to_problem(s) for s in specs]
        pool = api.Pool(sum(j3d.j3d_pool_request_bytes(p) for p in problems), max_slots=len(problems))
        if case["two_sweep"]:
            pool.set_two_sweep(True)
        return {"case": case, "pool": pool, "problems": problems, "iters": [s.iters for s in specs]}
    p = j3d.Problem(_n(case), (case["bx"], case["by"], case["bz"]), bc=_bc(seed))
    nbytes = j3d.j3d_field_bytes(p)
    u0 = _interior(case, seed)
    return {"case": case, "problem": p, "nbytes": nbytes, "u0": u0, "out": torch.empty_like(u0),
            "fields": torch.empty(nbytes, dtype=torch.uint8, device=DEV)}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "solve":
        s, left, residuals = state["solver"], case["iters"], []
        s.set_interior(state["u0"])
        while left > 0:
            k = min(left, case["check"] or left)
            residuals.append(s.run(k, mode=case["mode"], residual=True))
            left -= k
        return {"u": s.get_interior_device(), "residuals": residuals}
    if kind == "serial":
        with api.Solver(_n(case), seed=state["seed"]) as s:
            r = s.run(case["iters"], residual=True)
            return {"u": s.get_interior(), "residuals": [r]}
    if kind == "batch":
        with api.Batch(state["problems"], state["iters"]) as b:
            residuals = b.run(two_sweep=case["two_sweep"])
            us = []
            for i, p in enumerate(state["problems"]):
                u = torch.empty(p.n[::-1], dtype=torch.float64, device=DEV)
                j3d.j3d_batch_get_interior(b.h, i, u.data_ptr(), True)
                us.append(u)
        return {"u": us, "residuals": residuals}
    if kind == "pool":
        pool = state["pool"]
        slots = [pool.try_admit(p, it) for p, it in zip(state["problems"], state["iters"])]
        done = 0
        while done < len(slots):
            finished, busy = pool.poll()
            done += len(finished)
            if not busy and done < len(slots):
                pool.step(50)
        results = [pool.result(slot) for slot in slots]
        for slot in slots:
            pool.release(slot)
        return {"u": [r[0] for r in results], "residuals": [r[1] for r in results],
                "sweeps": [r[2] for r in results]}
    r = j3d.j3d_solve_noalloc(state["problem"], state["fields"].data_ptr(), state["nbytes"],
                              state["u0"].data_ptr(), state["out"].data_ptr(), case["iters"], True,
                              torch.cuda.current_stream().cuda_stream)
    return {"u": state["out"], "residuals": [r]}


# ---- what a pass cannot do without ----------------------------------------------

def work(case):
    """Bytes: the interior and boundary values that come in and the interior that
    goes out, once each.  Flops: six additions and a multiplication per update."""
    def one(n, iters, reads_interior):
        cells = n[0] * n[1] * n[2]
        shell = 2 * (n[0] * n[1] + n[1] * n[2] + n[0] * n[2])
        return (8 * cells * (2 if reads_interior else 1) + 8 * shell, 7 * cells * iters)

    if case["kind"] in ("batch", "pool"):
        parts = [one(s.n, s.iters, False) for s in _mix(case, 1)]
    else:
        parts = [one(_n(case), case["iters"], case["kind"] != "serial")]
    return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}


# ---- the same results from plain torch ------------------------------------------

def _seeded(n, seed, pid):
    """Uniform [0, 1) from SplitMix64: the problem's stream starts in the state
    that output pid + 1 of the generator's stream from `seed` gives."""
    mask = (1 << 64) - 1
    gamma, m1, m2 = 0x9E3779B97F4A7C15, 0xBF58476D1CE4E5B9, 0x94D049BB133111EB

    def signed(v):
        v &= mask
        return v - (1 << 64) if v >> 63 else v

    z = (seed + (pid + 1) * gamma) & mask
    z = ((z ^ (z >> 30)) * m1) & mask
    z = ((z ^ (z >> 27)) * m2) & mask
    s0 = z ^ (z >> 31)

    def shr(t, k):
        return (t >> k) & ((1 << (64 - k)) - 1)

    g = torch.arange(1, n[0] * n[1] * n[2] + 1, dtype=torch.int64, device=DEV)
    t = g * signed(gamma) + signed(s0)
    t = (t ^ shr(t, 30)) * signed(m1)
    t = (t ^ shr(t, 27)) * signed(m2)
    t = t ^ shr(t, 31)
    return (shr(t, 11).to(torch.float64) * 2.0 ** -53).reshape(n[2], n[1], n[0])


def _jacobi(u0, iters, faces, check=0):
    """Interior after `iters` sweeps and the residual of each checked sweep."""
    nz, ny, nx = u0.shape
    a = torch.zeros((nz + 2, ny + 2, nx + 2), dtype=torch.float64, device=u0.device)
    inner = (slice(1, -1),) * 3
    ring = [(inner[0], inner[1], 0), (inner[0], inner[1], -1), (inner[0], 0, inner[2]), (inner[0], -1, inner[2]),
            (0, inner[1], inner[2]), (-1, inner[1], inner[2])]
    for at, v in zip(ring, faces):
        a[at] = v if isinstance(v, float) else torch.as_tensor(v, device=u0.device)
    a[inner] = u0
    b = a.clone()
    s = torch.empty_like(u0)
    residuals = []
    for t in range(1, iters + 1):
        torch.add(a[inner], a[1:-1, 1:-1, :-2], out=s)
        s += a[1:-1, 1:-1, 2:]
        s += a[1:-1, :-2, 1:-1]
        s += a[1:-1, 2:, 1:-1]
        s += a[:-2, 1:-1, 1:-1]
        s += a[2:, 1:-1, 1:-1]
        s *= 1.0 / 7.0
        b[inner] = s
        if t == iters or (check and t % check == 0):
            s -= a[inner]
            residuals.append(float(s.abs_().max()))
        a, b = b, a
    return a[inner].clone(), residuals


def exact(case, seed):
    kind = case["kind"]
    if kind == "solve":
        bc = _bc(seed) if case["bc"] else (0.0,) * 6
        u, r = _jacobi(_interior(case, seed), case["iters"], _faces(case, seed) if case["faces"] else bc,
                       case["check"])
        return {"u": u, "residuals": r}
    if kind == "serial":
        u, r = _jacobi(_seeded(_n(case), seed, 0), case["iters"], (0.0,) * 6)
        return {"u": u.cpu().numpy(), "residuals": r}
    if kind == "noalloc":
        u, r = _jacobi(_interior(case, seed), case["iters"], _bc(seed))
        return {"u": u, "residuals": r}
    specs = _mix(case, seed)
    done = [_jacobi(_seeded(s.n, s.seed, s.pid), s.iters, s.bc) for s in specs]
    if kind == "batch":
        return {"u": [u for u, _ in done], "residuals": np.array([r[-1] for _, r in done])}
    return {"u": [u.cpu().numpy() for u, _ in done], "residuals": [r[-1] for _, r in done],
            "sweeps": [s.iters for s in specs]}
