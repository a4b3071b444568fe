"""Performance cases: the calls that a program using this framework makes, with the inputs it makes them on.

Every case goes through the Python entry points (``fr.route``, ``fr.accumulate``, ``fr.fill_depressions``,
``fr.FlowAccumulate``, ``fr.adjoint``, ``fr.Batch``).  The terrain is the benchmark's recipe made on the GPU: a
diamond-square fractal (Hurst 0.7) in [0, 1], a tilt of 0.01 per row (``tilted``; 0 for ``raw`` and ``filled``) and
U[0, 1e-3) noise, rounded once to float32; ``filled`` terrain is depression-filled before it is routed, as the
paper's workflow does.

Fields of a case: ``kind`` (what is called), ``rows``, ``cols``, and, where the kind has them, ``terrain``, ``rule``,
``dtype`` of the water, ``rain`` (drawn per cell, or unit), ``counts`` and ``mass``; a batch has ``tiles`` and the
range ``lo`` to ``hi`` of their sides.
"""
import math
import random

import torch

import paper_2606_12800_amd as fr

DEV = "cuda"
HURST, TILT, NOISE = 0.7, 0.01, 1e-3
# Neighbour k of a cell: row-major window order.
STEPS = [(-1, -1), (-1, 0), (-1, 1), (0, -1), (0, 1), (1, -1), (1, 0), (1, 1)]
DTYPES = {"f32": torch.float32, "f64": torch.float64, "none": None}
# Largest grids for which exact() stays within seconds.
EXACT_TREE_CELLS, EXACT_FILL_CELLS, EXACT_SPLIT_CELLS = 1 << 27, 1 << 22, 1 << 24


def listed():
    return [
        # Interactive use and tests: one small grid (the benchmark's 256^2 configuration), bound by launches.
        {"name": "d8_256", "kind": "route", "rows": 256, "cols": 256, "terrain": "tilted", "rule": "d8",
         "dtype": "f32", "rain": True, "counts": False, "mass": False},
        # One ordinary tilted DEM, all outputs (the benchmark's 4096^2 configuration).
        {"name": "d8_4096", "kind": "route", "rows": 4096, "cols": 4096, "terrain": "tilted", "rule": "d8",
         "dtype": "f32", "rain": True, "counts": True, "mass": True},
        # The headline workload's kind at 4.8e8 cells: a large tilted DEM, all outputs.
        {"name": "d8_20000x24000", "kind": "route", "rows": 20000, "cols": 24000, "terrain": "tilted", "rule": "d8",
         "dtype": "f32", "rain": True, "counts": True, "mass": True},
        # The paper's workflow on one DEM tile with odd sides: fill, receivers, water and drainage counts.
        {"name": "workflow_2047x1801", "kind": "workflow", "rows": 2047, "cols": 1801, "rule": "d8", "dtype": "f32",
         "rain": True, "counts": True, "mass": False},
        # Routing of a large depression-filled DEM: flow in every direction.
        {"name": "d8_filled_12000x9001", "kind": "route", "rows": 12000, "cols": 9001, "terrain": "filled",
         "rule": "d8", "dtype": "f32", "rain": True, "counts": True, "mass": True},
        # Drainage area and float64 water by the four-neighbour rule, ragged sides.
        {"name": "d4_f64_filled_1531x2111", "kind": "route", "rows": 1531, "cols": 2111, "terrain": "filled",
         "rule": "d4", "dtype": "f64", "rain": True, "counts": True, "mass": True},
        # Depression filling alone, a large DEM.
        {"name": "fill_8192", "kind": "fill", "rows": 8192, "cols": 8192, "rule": "d8"},
        # Multiple flow directions on a large tilted DEM (the benchmark's MFD workload, a quarter of its cells).
        {"name": "mfd_8192", "kind": "route", "rows": 8192, "cols": 8192, "terrain": "tilted", "rule": "mfd",
         "dtype": "f32", "rain": False, "counts": False, "mass": False},
        # Multiple flow directions on a filled DEM.
        {"name": "mfd_filled_2048", "kind": "route", "rows": 2048, "cols": 2048, "terrain": "filled", "rule": "mfd",
         "dtype": "f32", "rain": True, "counts": False, "mass": False},
        # A training step's flow layer: forward, and the gradient with respect to the rain.
        {"name": "grad_mfd_1200x1601", "kind": "grad", "rows": 1200, "cols": 1601, "terrain": "filled",
         "rule": "mfd", "dtype": "f32"},
        # Sensitivity of 64 gauges (the benchmark's adjoint configuration).
        {"name": "adjoint_mfd_4096", "kind": "adjoint", "rows": 4096, "cols": 4096, "terrain": "tilted",
         "rule": "mfd", "dtype": "f32"},
        # Serving: tiles of uneven size, D8 counts and MFD water by turns, as the benchmark's batch has them.
        {"name": "batch_48", "kind": "batch", "tiles": 48, "lo": 64, "hi": 2048, "shapes": 4},
    ]


def _sides(rng, lo, hi):
    """Rows and columns of a grid of lo to hi cells (log-uniform), up to four times as long as wide, often odd."""
    cells = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    aspect = math.exp(rng.uniform(math.log(0.5), math.log(2.0)))
    rows = max(3, int(math.sqrt(cells * aspect)))
    cols = max(3, int(math.sqrt(cells / aspect)))
    return {"rows": rows, "cols": cols}


def draw(rng):
    kind = rng.choice(["route", "route", "route", "workflow", "fill", "mfd", "mfd", "grad", "adjoint", "batch"])
    if kind == "route":
        dtype = rng.choice(["f32", "f32", "f64", "none"])
        return {"kind": "route", **_sides(rng, 1 << 12, 1 << 28), "terrain": rng.choice(["tilted", "filled", "raw"]),
                "rule": rng.choice(["d8", "d8", "d4"]), "dtype": dtype, "rain": rng.random() < 0.7,
                "counts": dtype == "none" or rng.random() < 0.6, "mass": dtype != "none" and rng.random() < 0.5}
    if kind == "workflow":
        return {"kind": "workflow", **_sides(rng, 1 << 12, 1 << 25), "rule": rng.choice(["d8", "d4"]),
                "dtype": rng.choice(["f32", "f64"]), "rain": rng.random() < 0.7, "counts": rng.random() < 0.6,
                "mass": rng.random() < 0.5}
    if kind == "fill":
        return {"kind": "fill", **_sides(rng, 1 << 12, 1 << 26), "rule": rng.choice(["d8", "d8", "d4"])}
    # Multiple directions and gradients: up to the benchmark's 4096^2 on tilted terrain, and smaller grids where water
    # runs every way.
    if kind == "mfd":
        terrain = rng.choice(["tilted", "filled", "raw"])
        return {"kind": "route", **_sides(rng, 1 << 12, 1 << (24 if terrain == "tilted" else 22)), "terrain": terrain,
                "rule": "mfd", "dtype": rng.choice(["f32", "f32", "f64"]), "rain": rng.random() < 0.5,
                "counts": False, "mass": rng.random() < 0.5}
    if kind in ("grad", "adjoint"):
        terrain = rng.choice(["tilted", "filled"])
        return {"kind": kind, **_sides(rng, 1 << 12, 1 << (24 if terrain == "tilted" else 20)), "terrain": terrain,
                "rule": rng.choice(["mfd", "mfd", "d8"]), "dtype": rng.choice(["f32", "f32", "f64"])}
    return {"kind": "batch", "tiles": rng.randint(4, 48), "lo": 64, "hi": rng.choice([512, 1024, 2048]),
            "shapes": rng.randint(0, 1 << 20)}


# ---------------------------------------------------------------------------
# Inputs

def _generator(seed, stream):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 64 + stream)


def _fractal(rows, cols, gen):
    """Diamond-square fractal, float64, normalised to [0, 1]."""
    k = max(1, math.ceil(math.log2(max(rows, cols, 3) - 1)))
    n = (1 << k) + 1
    a = torch.zeros((n, n), dtype=torch.float64, device=DEV)

    def u(h, w):
        return torch.rand((h, w), generator=gen, dtype=torch.float32, device=DEV).double().mul_(2.0).sub_(1.0)

    a[:: n - 1, :: n - 1] = u(2, 2)
    for level in range(1, k + 1):
        step = (n - 1) >> (level - 1)
        half, amp = step // 2, 2.0 ** (-HURST * level)
        c = a[::step, ::step]
        mid = (c[:-1, :-1] + c[:-1, 1:] + c[1:, :-1] + c[1:, 1:]) * 0.25
        mid += u(*mid.shape) * amp
        a[half::step, half::step] = mid
        for horizontal in (True, False):
            # Edge points between two corners: those, and the one or two centres beside them.
            c0, c1 = (c[:, :-1], c[:, 1:]) if horizontal else (c[:-1, :], c[1:, :])
            s = c0 + c1
            w = torch.full_like(s, 2.0)
            if horizontal:
                s[1:] += mid
                s[:-1] += mid
                w[1:] += 1.0
                w[:-1] += 1.0
            else:
                s[:, 1:] += mid
                s[:, :-1] += mid
                w[:, 1:] += 1.0
                w[:, :-1] += 1.0
            s /= w
            s += u(*s.shape) * amp
            if horizontal:
                a[::step, half::step] = s
            else:
                a[half::step, ::step] = s
    a = a[:rows, :cols].contiguous()
    lo, hi = a.min(), a.max()
    return a.sub_(lo).div_(hi - lo)


def _dem(case, seed, stream=0):
    rows, cols = case["rows"], case["cols"]
    a = _fractal(rows, cols, _generator(seed, stream))
    if case.get("terrain") == "tilted":
        a += TILT * torch.arange(rows, dtype=torch.float64, device=DEV)[:, None]
    a += NOISE * torch.rand((rows, cols), generator=_generator(seed, stream + 1), dtype=torch.float32, device=DEV)
    return a.float()


def _rain(case, seed):
    if not case.get("rain", True):
        return None
    dtype = DTYPES[case["dtype"]] or torch.float32
    # 24 random bits: exact in float32.
    return torch.rand((case["rows"], case["cols"]), generator=_generator(seed, 8), dtype=torch.float32,
                      device=DEV).to(dtype)


def _gauges(case, seed):
    """64 weights at cells of the grid (fewer on a tiny one), as a field of zeros elsewhere."""
    cells = case["rows"] * case["cols"]
    g = _generator(seed, 9)
    at = torch.randint(0, cells, (64,), generator=g, device=DEV)
    w = torch.randn(64, generator=g, dtype=torch.float64, device=DEV)
    qbar = torch.zeros(cells, dtype=DTYPES[case["dtype"]], device=DEV)
    qbar[at] = w.to(qbar.dtype)
    return qbar.view(case["rows"], case["cols"])


def _loss(case, seed):
    """Gradient of a loss with respect to the water at every cell."""
    return torch.randn((case["rows"], case["cols"]), generator=_generator(seed, 10), dtype=torch.float32,
                       device=DEV).to(DTYPES[case["dtype"]])


def _tile_cases(case):
    """Shapes of the batch: D8 counts and MFD water by turns, on tilted terrain."""
    rng = random.Random(case["shapes"])
    return [{"rows": rng.randint(case["lo"], case["hi"]), "cols": rng.randint(case["lo"], case["hi"]),
             "terrain": "tilted", "rule": "mfd" if i % 2 else "d8"} for i in range(case["tiles"])]


def _tile_dems(case, seed):
    return [_dem(t, seed * 1000 + i) for i, t in enumerate(_tile_cases(case))]


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        tiles = []
        for t, z in zip(_tile_cases(case), _tile_dems(case, seed)):
            if t["rule"] == "mfd":
                tiles.append({"z": z, "rule": "mfd", "q": torch.empty_like(z)})
            else:
                tiles.append({"z": z, "rule": "d8", "counts": torch.empty(z.shape, dtype=torch.int64, device=DEV)})
        return {"case": case, "tiles": tiles, "batch": fr.Batch(tiles)}
    z = _dem(case, seed)
    if case.get("terrain") == "filled":
        z = fr.fill_depressions(z, case["rule"])
    s = {"case": case, "z": z}
    if kind in ("route", "workflow"):
        s["rain"] = _rain(case, seed)
    elif kind == "grad":
        s["rain"] = _rain(case, seed)
        s["loss"] = _loss(case, seed)
    elif kind == "adjoint":
        s["code"] = fr.receivers(z, case["rule"])
        s["qbar"] = _gauges(case, seed)
    return s


def run(state):
    c = state["case"]
    kind = c["kind"]
    if kind in ("route", "workflow"):
        z = state["z"] if kind == "route" else fr.fill_depressions(state["z"], c["rule"])
        code, q, counts, mass = fr.route(z, state["rain"], c["rule"], DTYPES[c["dtype"]], counts=c["counts"],
                                         mass=c["mass"])
        # Counts as signed integers (a view): torch indexes no unsigned 64-bit tensors.
        out = (code, q, None if counts is None else counts.view(torch.int64), mass)
        return out if kind == "route" else (z,) + out
    if kind == "fill":
        return fr.fill_depressions(state["z"], c["rule"])
    if kind == "grad":
        rain = state["rain"].detach().requires_grad_(True)
        q = fr.FlowAccumulate.apply(rain, state["z"], c["rule"])
        (grad,) = torch.autograd.grad(q, rain, state["loss"])
        return q.detach(), grad
    if kind == "adjoint":
        z = state["z"] if c["rule"] == "mfd" else None
        return fr.adjoint(state["code"], state["qbar"], z, c["rule"])
    state["batch"].run()
    return [t["q"] if "q" in t else t["counts"] for t in state["tiles"]]


def work(case):
    """Arrays of the call read or written once each; about 30 operations a cell and neighbour set."""
    kind = case["kind"]
    if kind == "batch":
        cells = [(t["rows"] * t["cols"], t["rule"]) for t in _tile_cases(case)]
        return {"bytes": sum(n * (8 if r == "mfd" else 12) for n, r in cells), "flops": 40 * sum(n for n, _ in cells)}
    n = case["rows"] * case["cols"]
    if kind == "fill":
        return {"bytes": 8 * n, "flops": 10 * n}
    size = {"f32": 4, "f64": 8, "none": 0}[case["dtype"]]
    if kind == "grad":
        return {"bytes": n * (4 + 4 * size), "flops": 80 * n}
    if kind == "adjoint":
        return {"bytes": n * (1 + 2 * size + (4 if case["rule"] == "mfd" else 0)), "flops": 40 * n}
    per = 4 + 1 + size + (max(size, 4) if case["rain"] else 0) + (8 if case["counts"] else 0)
    if kind == "workflow":
        per += 8
    return {"bytes": per * n, "flops": 40 * n}


# ---------------------------------------------------------------------------
# The same results from plain torch in 64 bits

def _shifted(a, k, fill):
    """a's neighbour k of every cell, `fill` off the grid."""
    dr, dc = STEPS[k]
    out = torch.full_like(a, fill)
    rows, cols = a.shape
    r0, r1, c0, c1 = max(0, -dr), rows - max(0, dr), max(0, -dc), cols - max(0, dc)
    out[r0:r1, c0:c1] = a[r0 + dr:r1 + dr, c0 + dc:c1 + dc]
    return out


def _fill(z, rule):
    """The filled surface: float32 steps counted in the order-preserving integer keys of the elevations."""
    bits = (z + 0.0).view(torch.int32).long()
    key = torch.where(bits >= 0, bits, -(bits & 0x7FFFFFFF))
    big = 1 << 40
    f = torch.full_like(key, big)
    edge = torch.zeros_like(key, dtype=torch.bool)
    edge[0], edge[-1], edge[:, 0], edge[:, -1] = True, True, True, True
    f[edge] = key[edge]
    inside, zin = f[1:-1, 1:-1], key[1:-1, 1:-1]
    rows, cols = f.shape
    ks = range(8) if rule != "d4" else (1, 3, 4, 6)
    while rows > 2 and cols > 2:
        before = f.clone()
        for _ in range(64):
            low = None
            for k in ks:
                dr, dc = STEPS[k]
                v = f[1 + dr:rows - 1 + dr, 1 + dc:cols - 1 + dc]
                low = v.clone() if low is None else torch.minimum(low, v)
            torch.minimum(inside, torch.maximum(zin, low + 1), out=low)
            inside.copy_(low)
        if torch.equal(before, f):
            break
    out = torch.where(f >= 0, f, (-f) | 0x80000000)
    return torch.where(out >= 1 << 31, out - (1 << 32), out).int().view(torch.float32)


def _receivers(z, rule):
    """Steepest strictly lower neighbour by float32 slopes, ties to the lowest k; its cell, or the cell count at a
    sink."""
    rows, cols = z.shape
    diag = torch.tensor(0x3F3504F3, dtype=torch.int32, device=z.device).view(torch.float32)
    best = torch.zeros_like(z)
    to = torch.full(z.shape, z.numel(), dtype=torch.int64, device=z.device)
    at = torch.arange(z.numel(), device=z.device).view(rows, cols)
    for k in (range(8) if rule == "d8" else (1, 3, 4, 6)):
        dr, dc = STEPS[k]
        s = z - _shifted(z, k, math.inf)
        if dr and dc:
            s = s * diag
        better = s > best
        best = torch.where(better, s, best)
        to = torch.where(better, at + (dr * cols + dc), to)
    return to.view(-1)


def _tree_sums(to, x):
    """Sums of x over each cell and all cells that drain through it, by pointer doubling."""
    n = to.numel()
    to = torch.cat([to, torch.tensor([n], device=to.device)])
    q, live = x, torch.nonzero(to[:-1] < n).view(-1)
    while live.numel():
        q = q.index_add(0, to[live], q[live])
        to = to[to]
        live = live[to[live] < n]
    return q


def _path_sums(to, x):
    """Sums of x over each cell's flow path (the transpose of _tree_sums)."""
    n = to.numel()
    to = torch.cat([to, torch.tensor([n], device=to.device)])
    y = torch.cat([x, x.new_zeros(1)])
    while bool((to[:-1] < n).any()):
        y = y + y[to]
        to = to[to]
    return y[:-1]


def _fractions(z, p=1.1):
    """Receivers [8, n] (the cell itself where there is none) and fractions [8, n] of the multiple-direction rule."""
    rows, cols = z.shape
    zd = z.double()
    at = torch.arange(z.numel(), device=z.device).view(rows, cols)
    to, f = [], []
    for k, (dr, dc) in enumerate(STEPS):
        s = ((zd - _shifted(zd, k, math.inf)) / (math.sqrt(2.0) if dr and dc else 1.0)).clamp_(min=0.0)
        f.append(s.view(-1))
        to.append(torch.where(s > 0, at + (dr * cols + dc), at).view(-1))
    f = torch.stack(f)
    top = f.max(0).values
    f = (f / torch.where(top > 0, top, 1.0)) ** p
    total = f.sum(0)
    return torch.stack(to), f / torch.where(total > 0, total, 1.0)


def _split_levels(to):
    """Cells in levels: each after all cells that give it water."""
    n = to.shape[1]
    at = torch.arange(n, device=to.device)
    waits = torch.zeros(n, dtype=torch.int32, device=to.device)
    for k in range(8):
        waits.index_add_(0, to[k], (to[k] != at).int())
    mark = torch.empty(n, dtype=torch.int32, device=to.device)
    front = torch.nonzero(waits == 0).view(-1)
    while front.numel():
        yield front
        nb = to[:, front]
        real = nb != front
        nb, real = nb.reshape(-1), real.reshape(-1)
        waits.index_add_(0, nb, -real.int())
        ready = nb[real & (waits[nb] == 0)]
        order = torch.arange(ready.numel(), dtype=torch.int32, device=to.device)
        mark[ready] = order
        front = ready[mark[ready] == order]


def _split_forward(to, f, x):
    q = x.clone()
    for front in _split_levels(to):
        q.index_add_(0, to[:, front].reshape(-1), (f[:, front] * q[front]).reshape(-1))
    return q


def _split_adjoint(to, f, x):
    y = x.clone()
    for front in reversed(list(_split_levels(to))):
        y[front] = x[front] + (f[:, front] * y[to[:, front]]).sum(0)
    return y


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        cases, dems = _tile_cases(case), _tile_dems(case, seed)
        split = [z for t, z in zip(cases, dems) if t["rule"] == "mfd"]
        tos, fs, at = [], [], 0
        total = sum(z.numel() for z in split)
        for z in split:
            to, f = _fractions(z)
            tos.append(to + at)
            fs.append(f)
            at += z.numel()
        to, f = torch.cat(tos, 1), torch.cat(fs, 1)
        del tos, fs
        q = iter(_split_forward(to, f, torch.ones(total, dtype=torch.float64, device=DEV)).split(
            [z.numel() for z in split]))
        return [next(q).view(z.shape) if t["rule"] == "mfd" else None for t, z in zip(cases, dems)]
    n = case["rows"] * case["cols"]
    split = case["rule"] == "mfd"
    filled = kind in ("fill", "workflow") or case.get("terrain") == "filled"
    if n > (EXACT_SPLIT_CELLS if split else EXACT_TREE_CELLS) or (filled and n > EXACT_FILL_CELLS):
        return None
    z = _dem(case, seed)
    if filled:
        z = _fill(z, case["rule"])
    if kind == "fill":
        return z.double()
    if split:
        to, f = _fractions(z)
    else:
        to = _receivers(z, case["rule"])
    forward = (lambda x: _split_forward(to, f, x)) if split else (lambda x: _tree_sums(to, x))
    adjoint = (lambda x: _split_adjoint(to, f, x)) if split else (lambda x: _path_sums(to, x))
    if kind == "adjoint":
        return adjoint(_gauges(case, seed).double().view(-1)).view(z.shape)
    rain = _rain(case, seed)
    x = torch.ones(n, dtype=torch.float64, device=DEV) if rain is None else rain.double().view(-1)
    if kind == "grad":
        loss = _loss(case, seed).double().view(-1)
        return forward(x).view(z.shape), adjoint(loss).view(z.shape)
    if case["dtype"] == "none":
        return None
    q = forward(x)
    mass = None
    if case["mass"]:
        sink = (to == torch.arange(n, device=DEV)).all(0) if split else to == n
        mass = torch.stack([q[sink].sum(), x.sum()])
    out = (None, q.view(z.shape), None, mass)
    return (z.double(),) + out if kind == "workflow" else out
