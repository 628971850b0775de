"""Cases by which the solver's speed is judged, through its public Python entry points.

Matrices are built on the GPU with torch, in the numbering and with the values
of workloads/gen.py: Dirichlet box stencils with x varying fastest (5-point
2-D, 7-point 3-D, 125-point 3-D, and the 27-point stencil with one lognormal
weight per edge) and random sparse SPD matrices.  The exact solution is
uniform and b = A x*, so every seed is another system of equations;
a solve returns x, the iteration count and the status.
"""

import math
import random
import types

import torch

from paper_2105_06176_amd import ppcg

DEV = "cuda"


# ---------------------------------------------------------------- the cases
def listed():
    return [
        # smallest: one 2-D system of 4,096 rows, where latency decides
        {"name": "solve_2d_64", "kind": "2d", "nx": 64, "ny": 64, "tol": 1e-8},
        # ordinary 2-D system of odd size, a few hundred short iterations
        {"name": "solve_2d_301", "kind": "2d", "nx": 301, "ny": 301, "tol": 1e-6},
        # the benchmark's grid, solved to its tolerance
        {"name": "solve_3d_128", "kind": "3d", "nx": 128, "ny": 128, "nz": 128, "tol": 1e-10},
        # classic PCG on a box of unequal odd sides, from an initial guess
        {"name": "pcg_3d_odd", "kind": "pcg", "nx": 97, "ny": 131, "nz": 75, "tol": 1e-8},
        # variable coefficients: no value repeats, the matrix is most of the bytes
        {"name": "stencil27_160", "kind": "s27", "nx": 160, "ny": 160, "nz": 160, "iters": 30},
        # long rows, constant coefficients, stopped by the preconditioned norm
        {"name": "stencil125_165", "kind": "s125", "nx": 165, "ny": 165, "nz": 165, "tol": 1e-5},
        # columns without locality: a large matrix, and one that fits the caches
        {"name": "random_4096000", "kind": "random", "n": 4096000, "draws": 8, "tol": 1e-10},
        {"name": "random_259789", "kind": "random", "n": 259789, "draws": 8, "tol": 1e-10},
        # FP32 values and vectors with FP64 reliable updates, to a tolerance only FP64 reaches
        {"name": "mixed_s27_128", "kind": "mixed", "nx": 128, "ny": 128, "nz": 128, "tol": 1e-10},
        # many systems of one kind and uneven size in one call (e.g. implicit time steps)
        {"name": "batch_64", "kind": "batch", "count": 64, "lo": 32, "hi": 512, "spec": 0, "tol": 1e-10},
        # a small batch of small systems
        {"name": "batch_8_small", "kind": "batch", "count": 8, "lo": 24, "hi": 120, "spec": 5, "tol": 1e-8},
        # a burst of requests to the server, matrices and right-hand sides on the host
        {"name": "serve_12", "kind": "serve", "count": 12, "nlo": 1000, "nhi": 120000, "spec": 3},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["2d", "2d", "3d", "3d", "pcg", "s27", "s125", "random", "random", "mixed", "batch", "serve"])
    if kind == "2d":
        nx = _log(rng, 20, 320)
        ny = min(320, max(20, int(nx * rng.uniform(0.7, 1.4))))
        return {"kind": kind, "nx": nx, "ny": ny, "tol": rng.choice([1e-6, 1e-8]) if nx * ny <= 20000 else 1e-6}
    if kind in ("3d", "pcg"):
        return {"kind": kind, "nx": _log(rng, 18, 144), "ny": _log(rng, 18, 144), "nz": _log(rng, 18, 128),
                "tol": rng.choice([1e-6, 1e-8, 1e-10])}
    if kind == "s27":
        return {"kind": kind, "nx": _log(rng, 20, 160), "ny": _log(rng, 20, 160), "nz": _log(rng, 20, 160),
                "iters": rng.randint(8, 30)}
    if kind == "s125":
        return {"kind": kind, "nx": _log(rng, 16, 165), "ny": _log(rng, 16, 165), "nz": _log(rng, 16, 165), "tol": 1e-5}
    if kind == "random":
        n = _log(rng, 4000, 4096000)
        return {"kind": kind, "n": n, "draws": 8 if n > 1400000 else rng.choice([8, 23]), "tol": rng.choice([1e-8, 1e-10])}
    if kind == "mixed":
        return {"kind": kind, "nx": _log(rng, 40, 128), "ny": _log(rng, 40, 128), "nz": _log(rng, 40, 128), "tol": 1e-10}
    if kind == "batch":
        lo = _log(rng, 20, 60)
        return {"kind": kind, "count": _log(rng, 3, 60), "lo": lo, "hi": _log(rng, 2 * lo, 512),
                "spec": rng.randrange(1 << 20), "tol": rng.choice([1e-8, 1e-10])}
    return {"kind": "serve", "count": rng.randint(3, 12), "nlo": 1000, "nhi": _log(rng, 10000, 120000),
            "spec": rng.randrange(1 << 20)}


# ---------------------------------------------------------------- matrices
def _generator(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _offsets(points):
    """Stencil offsets (dx, dy, dz) in ascending linear order."""
    if points in (27, 125):
        r = 1 if points == 27 else 2
        span = range(-r, r + 1)
        return [(dx, dy, dz) for dz in span for dy in span for dx in span]
    star = [(0, -1, 0), (-1, 0, 0), (0, 0, 0), (1, 0, 0), (0, 1, 0)]
    return star if points == 5 else [(0, 0, -1)] + star + [(0, 0, 1)]


def _grid(dims, points):
    """(columns [n, K], inside-the-grid mask [n, K], offsets, their linear offsets)."""
    nx, ny, nz = dims
    offs = _offsets(points)
    lin = [dx + nx * (dy + ny * dz) for dx, dy, dz in offs]
    idx = torch.arange(nx * ny * nz, dtype=torch.int32, device=DEV)
    x, y, z = idx % nx, idx // nx % ny, idx // (nx * ny)
    ok = torch.empty(idx.numel(), len(offs), dtype=torch.bool, device=DEV)
    for k, (dx, dy, dz) in enumerate(offs):
        ok[:, k] = ((x + dx >= 0) & (x + dx < nx) & (y + dy >= 0) & (y + dy < ny) & (z + dz >= 0) & (z + dz < nz))
    cols = idx[:, None] + torch.tensor(lin, dtype=torch.int32, device=DEV)[None, :]
    return cols, ok, offs, lin


def _row_ptr(lengths):
    rp = torch.zeros(lengths.numel() + 1, dtype=torch.int32, device=DEV)
    rp[1:] = torch.cumsum(lengths, 0)
    return rp


def _constant_stencil(dims, points, diag):
    cols, ok, offs, _ = _grid(dims, points)
    vals = torch.full((len(offs),), -1.0, dtype=torch.float64, device=DEV)
    vals[offs.index((0, 0, 0))] = diag
    rp = _row_ptr(ok.sum(1))
    return rp, cols[ok], vals[None, :].expand_as(cols)[ok]


def _lognormal27(dims, seed, shift=1e-3):
    cols, ok, offs, lin = _grid(dims, 27)
    n = cols.shape[0]
    g = _generator(seed)
    vals = torch.zeros(n, 27, dtype=torch.float64, device=DEV)
    for k, d in enumerate(lin):
        if d > 0:
            w = torch.exp(torch.randn(n, dtype=torch.float64, device=DEV, generator=g))
            vals[:, k] = -w
            vals[d:, 26 - k] = -w[: n - d]  # the edge's other end: offset -d
    vals *= ok
    vals[:, 13] = -vals.sum(1) + shift
    return _row_ptr(ok.sum(1)), cols[ok], vals[ok]


def _random_spd(n, draws, seed, dominance=1e-2):
    g = _generator(seed)
    rows = torch.arange(n, device=DEV).repeat_interleave(draws)
    cols = torch.randint(0, n - 1, (n * draws,), device=DEV, generator=g)
    cols += cols >= rows
    key = torch.unique(torch.minimum(rows, cols) * n + torch.maximum(rows, cols))
    lo, hi = key // n, key % n
    v = torch.rand(key.numel(), dtype=torch.float64, device=DEV, generator=g) - 1.0
    diag = torch.arange(n, device=DEV)
    key = torch.cat([lo * n + hi, hi * n + lo, diag * (n + 1)])
    key, order = torch.sort(key)
    val = torch.cat([v, v, torch.zeros(n, dtype=torch.float64, device=DEV)])[order]
    row, col = key // n, (key % n).to(torch.int32)
    lengths = torch.bincount(row, minlength=n)
    val[row == key % n] = dominance - torch.segment_reduce(val, "sum", lengths=lengths)
    return _row_ptr(lengths), col, val


def _apply(A, x):
    """A x, each row summed in its stored order."""
    rp, ci, val = A
    return torch.segment_reduce(val * x[ci.long()], "sum", lengths=(rp[1:] - rp[:-1]).long())


def _xstar(n, seed):
    return 2.0 * torch.rand(n, dtype=torch.float64, device=DEV, generator=_generator(seed)) - 1.0


def _shifted2d(side, sigma):
    rp, ci, val = _constant_stencil((side, side, 1), 5, 4.0 + sigma)
    return rp, ci, val


def _specs(case):
    """Sizes of a batch's or a server burst's systems (part of the case, not of the inputs)."""
    rng = random.Random(case["spec"])
    if case["kind"] == "batch":
        return [(rng.randint(case["lo"], case["hi"]), rng.uniform(0.01, 0.5)) for _ in range(case["count"])]
    out = []
    for _ in range(case["count"]):
        n = math.exp(rng.uniform(math.log(case["nlo"]), math.log(case["nhi"])))
        out.append((rng.choices(["2d", "3d", "random"], [4, 3, 3])[0], int(n), rng.choice([1e-6, 1e-8])))
    return out


def _request(kind, n, seed):
    if kind == "2d":
        return _shifted2d(max(8, round(n ** 0.5)), 0.0)
    if kind == "3d":
        m = max(4, round(n ** (1 / 3)))
        return _constant_stencil((m, m, m), 7, 6.0)
    return _random_spd(max(64, n), 8, seed)


def _matrix(case, seed):
    kind = case["kind"]
    if kind == "random":
        return _random_spd(case["n"], case["draws"], seed)
    dims = (case["nx"], case["ny"], case.get("nz", 1))
    if kind in ("s27", "mixed"):
        return _lognormal27(dims, seed)
    points, diag = {"2d": (5, 4.0), "3d": (7, 6.0), "pcg": (7, 6.0), "s125": (125, 124.0)}[kind]
    return _constant_stencil(dims, points, diag)


def _systems(case, seed):
    """[(A, b, x0 or None, tol)] of the case, made from the seed."""
    if case["kind"] == "batch":
        mats = [(_shifted2d(s, sh), case["tol"]) for s, sh in _specs(case)]
    elif case["kind"] == "serve":
        mats = [(_request(k, n, seed * 1000 + i), tol) for i, (k, n, tol) in enumerate(_specs(case))]
    else:
        mats = [(_matrix(case, seed), case.get("tol", 0.0))]
    out = []
    for i, (A, tol) in enumerate(mats):
        n = A[0].numel() - 1
        xs = _xstar(n, seed * 7919 + i + 1)
        if case["kind"] == "s125":
            xs *= math.sqrt(3.0 / n)  # norm 1: the scale that the absolute tolerance is meant for
        x0 = xs + 0.1 * _xstar(n, seed * 7919 + 500 + i) if case["kind"] == "pcg" else None
        out.append((A, _apply(A, xs), x0, tol))
    return out


# ---------------------------------------------------------------- preparation and one pass
def _options(case):
    if case["kind"] == "s27":
        return {"fixed_iters": case["iters"]}
    opt = {"tol": case["tol"], "max_iter": 20000}
    if case["kind"] == "s125":
        opt["stop"] = "abs"
    elif case["kind"] == "pcg":
        opt["method"] = "pcg"
    elif case["kind"] == "mixed":
        opt["precision"] = "mixed"
    return opt


def _host(A):
    rp, ci, val = (t.cpu().numpy() for t in A)
    return types.SimpleNamespace(n=rp.size - 1, rp=rp, ci=ci, val=val)


def prepare(case, seed):
    systems = _systems(case, seed)
    if case["kind"] == "serve":
        reqs = [(_host(A), b.cpu().numpy(), tol) for A, b, _, tol in systems]
        return {"kind": "serve", "server": ppcg.Server(borrow=True), "reqs": reqs}
    torch.cuda.synchronize()  # the solvers read the matrices on streams of their own
    solvers = [ppcg.Solver(A, **_options(case)) for A, _, _, _ in systems]
    bs = [b for _, b, _, _ in systems]
    return {"kind": case["kind"], "solvers": solvers, "bs": bs, "x0": systems[0][2],
            "outs": [torch.empty_like(b) for b in bs]}


def _serve(server, reqs):
    """Submit every request, run the server until all are done, collect the solutions."""
    ids = [server.submit(A, b, tol, "auto") for A, b, tol in reqs]
    got = {}
    while len(got) < len(ids):
        active, queued = server.step()
        if len(ids) - len(got) > active + queued:
            for i, rid in enumerate(ids):
                if i not in got:
                    r = server.poll(rid)
                    if r is not None:
                        got[i] = r
    return [got[i] for i in range(len(ids))]


def run(state):
    if state["kind"] == "serve":
        done = _serve(state["server"], state["reqs"])
        return {"x": [x for x, _ in done], "status": [info["status"] for _, info in done]}
    if state["kind"] == "batch":
        xs, infos = ppcg.solve_batch(state["solvers"], state["bs"], outs=state["outs"])
        # 64 arrays at most are compared, so the solutions come as one
        return {"x": torch.cat(xs), "iters": torch.tensor([i["iters"] for i in infos]),
                "status": torch.tensor([i["status"] for i in infos])}
    x, info = state["solvers"][0].solve(state["bs"][0], x0=state["x0"], out=state["outs"][0])
    return {"x": x, "iters": info["iters"], "status": info["status"]}


# ---------------------------------------------------------------- what a pass cannot do without
def _iterations(kind, dims, tol):
    """About how many iterations a solve takes, as counted on such matrices (grids: per point of the longest side)."""
    if kind == "random":
        return 24 * math.log(tol) / math.log(1e-10)
    per_side = {"2d": {1e-6: 1.0, 1e-8: 2.2, 1e-10: 2.8}, "3d": {1e-6: 0.9, 1e-8: 1.6, 1e-10: 3.2},
                "mixed": {1e-10: 4.5}, "s125": {1e-5: 0.22}, "s27": {0.0: 1.0}}
    return per_side["3d" if kind == "pcg" else kind][tol] * max(dims)


def _iteration_work(kind, n, nnz):
    """Bytes and operations of one iteration: a matrix whose values all differ is read once (8-byte values, 4-byte
    columns; 4-byte values and no columns for the FP32 stencil), one of a few constants needs nothing but the
    stencil; of the vectors x, r, p and s and w = A u are read and written once (FP32 ones in the mixed mode, which
    iterates with three)."""
    per_entry = {"random": 12.0, "s27": 8.0, "mixed": 4.0}.get(kind, 0.0)
    per_row = 32.0 if kind == "mixed" else 64.0 if kind == "pcg" else 80.0
    return per_entry * nnz + per_row * n, 2.0 * nnz + 24.0 * n


def _sizes(case):
    """[(kind, n, nnz, iterations)] of the case's systems."""
    pts = {"2d": 5, "3d": 7, "pcg": 7, "s27": 27, "mixed": 27, "s125": 125}

    def one(kind, dims, n, tol, draws=8):
        if kind == "random":
            nnz = (2 * draws + 1) * n
        elif pts[kind] in (27, 125):
            r = 3 if pts[kind] == 27 else 5
            nnz = math.prod(r * d - (2 if r == 3 else 6) for d in dims)
        else:
            nnz = pts[kind] * n - 2 * sum(n // d for d in dims if d > 1)
        return kind, n, nnz, case.get("iters") or _iterations(kind, dims, tol)

    if case["kind"] == "batch":
        return [one("2d", (s, s, 1), s * s, case["tol"])[:3] + (min(3.3 * s, 30 / sh ** 0.5),) for s, sh in _specs(case)]
    if case["kind"] == "serve":
        out = []
        for kind, n, tol in _specs(case):
            m = round(n ** (1 / 2 if kind == "2d" else 1 / 3))
            dims = (m, m, 1) if kind == "2d" else (m, m, m)
            out.append(one(kind, dims, n if kind == "random" else math.prod(dims), tol))
        return out
    if case["kind"] == "random":
        return [one("random", (1, 1, 1), case["n"], case["tol"], case["draws"])]
    dims = (case["nx"], case["ny"], case.get("nz", 1))
    return [one(case["kind"], dims, math.prod(dims), case.get("tol", 0.0))]


def work(case):
    total = [0.0, 0.0]
    for kind, n, nnz, iters in _sizes(case):
        b, f = _iteration_work(kind, n, nnz)
        total[0] += iters * b + 16.0 * n
        total[1] += iters * f
    return {"bytes": total[0], "flops": total[1]}


# ---------------------------------------------------------------- the same in plain torch
def _conjugate_gradients(A, b, x0, tol, stop_abs, fixed):
    rp, ci, val = A
    n = b.numel()
    lengths = (rp[1:] - rp[:-1]).long()
    cols = ci.long()
    rows = torch.arange(n, device=DEV).repeat_interleave(lengths)
    dinv = torch.empty_like(b)
    on = cols == rows
    dinv[rows[on]] = 1.0 / val[on]
    del rows, on

    def apply(v):
        return torch.segment_reduce(val * v[cols], "sum", lengths=lengths)

    x = torch.zeros_like(b) if x0 is None else x0.clone()
    r = b.clone() if x0 is None else b - apply(x)
    bn = float(b.norm())
    p, gamma = None, 0.0
    for k in range(20000):
        u = dinv * r
        if fixed:
            done = k >= fixed
        else:
            done = float(u.norm()) < tol if stop_abs else float(r.norm()) <= tol * bn
        if done:
            break
        g = torch.dot(r, u)
        p = u if p is None else u + (g / gamma) * p
        s = apply(p)
        alpha = g / torch.dot(p, s)
        x = x + alpha * p
        r = r - alpha * s
        gamma = g
    return x


def exact(case, seed):
    xs = [_conjugate_gradients(A, b, x0, tol, case["kind"] == "s125", case.get("iters", 0))
          for A, b, x0, tol in _systems(case, seed)]
    if case["kind"] == "serve":
        return {"x": [x.cpu().numpy() for x in xs], "status": None}
    return {"x": torch.cat(xs), "iters": None, "status": None}
