"""Timed cases of the framework: the work its users have it do, through the public calls.

Every case is a program over one context (or a batch, or a server): option
pricing, stencil sweeps, Krylov and multigrid solves on assembled matrices,
a broadcast normalisation of a table, many solves in one persistent launch,
and a closed-loop client of the solve server.  Inputs are made on the GPU
from the seed; plans, compiled passes and recorded graphs are made in
prepare(), where such a program makes them once.
"""
import math

import numpy as np
import torch

import paper_2406_18109_amd as dfx

RATE, VOL = 0.02, 0.3
TORCH = {"f64": torch.float64, "f32": torch.float32}


def listed():
    return [
        # a pricing call on a handful of options: the smallest call a program
        # makes, submits and one launch
        {"name": "price_f64_1000", "kind": "price", "n": 1000, "dtype": "f64", "jit": 1},
        # the batch of the framework's headline benchmark
        {"name": "price_f64_2e26", "kind": "price", "n": 1 << 26, "dtype": "f64", "jit": 1},
        # single precision, a count that fills no tile evenly
        {"name": "price_f32_50000003", "kind": "price", "n": 50000003, "dtype": "f32", "jit": 1},
        # stencil sweeps on the benchmark's grid
        {"name": "sweep_8192", "kind": "sweep", "N": 8192, "sweeps": 4, "jit": 1},
        # an odd grid: every second row starts inside a 16-byte word
        {"name": "sweep_4099", "kind": "sweep", "N": 4099, "sweeps": 4, "jit": 1},
        # a table centred and scaled per column, weighted per row, with its
        # sum of squares: broadcasts along both axes, ragged width
        {"name": "table_f32_50021x1001", "kind": "table", "rows": 50021, "cols": 1001, "dtype": "f32", "jit": 1},
        # a small solve replayed from a graph, the paper's 100 iterations
        {"name": "cg_64x64", "kind": "cg", "m": 64, "dim": 2, "iters": 100, "graph": 1, "jit": 1},
        # the large solve of the benchmark
        {"name": "cg_256x256x256", "kind": "cg", "m": 256, "dim": 3, "iters": 8, "graph": 1, "jit": 1},
        # a nonsymmetric solve of ordinary size, side no multiple of the tiling
        {"name": "bicgstab_150x150x150", "kind": "bicgstab", "m": 150, "dim": 3, "iters": 8, "graph": 1, "jit": 1},
        # multigrid-preconditioned CG on the benchmark's hierarchy
        {"name": "gmg_1023", "kind": "gmg", "m": 1023, "levels": 9, "iters": 4, "graph": 1, "jit": 1},
        # independent solves of uneven sizes as streams of one persistent launch
        {"name": "batch_32_solves", "kind": "batch", "count": 32, "lo": 32, "hi": 256},
        # a client of the solve server: requests submitted at once, answers read back
        {"name": "serve_48_requests", "kind": "serve", "count": 48, "lo": 32, "hi": 256},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["price", "price", "sweep", "table", "cg", "cg", "bicgstab", "gmg", "batch", "serve"])
    jit = rng.choice([0, 1, 1])
    if kind == "price":
        return {"kind": kind, "n": _log(rng, 500, 1 << 26), "dtype": rng.choice(["f64", "f32"]), "jit": jit}
    if kind == "sweep":
        return {"kind": kind, "N": _log(rng, 130, 8192), "sweeps": rng.choice([2, 3, 4]), "jit": jit}
    if kind == "table":
        return {"kind": kind, "rows": _log(rng, 300, 50021), "cols": _log(rng, 33, 1030),
                "dtype": rng.choice(["f64", "f32"]), "jit": jit}
    if kind in ("cg", "bicgstab"):
        dim = rng.choice([2, 3])
        big = 1024 if dim == 2 else (256 if kind == "cg" else 160)
        m = _log(rng, 32, big)
        return {"kind": kind, "m": m, "dim": dim, "iters": rng.randint(4, 8), "graph": rng.choice([0, 1, 1]), "jit": jit}
    if kind == "gmg":
        lev = rng.choice([5, 6, 7, 8, 9])
        return {"kind": kind, "m": (2 << lev) - 1, "levels": lev - rng.choice([0, 1]), "iters": rng.randint(1, 4),
                "graph": rng.choice([0, 1]), "jit": jit}
    lo = _log(rng, 24, 64)
    return {"kind": kind, "count": rng.randint(4, 32), "lo": lo, "hi": lo + rng.randint(40, 180)}


# ---------------------------------------------------------------- inputs
def _gen(seed, k=0):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 64 + k)


def _uniform(n, lo, hi, dtype, seed, k):
    return (torch.rand(n, generator=_gen(seed, k), device="cuda", dtype=torch.float64) * (hi - lo) + lo).to(dtype)


def _stencil_csr(m, dim, conv=0.0):
    """CSR of the Poisson matrix of an m^dim grid (x fastest, Dirichlet rows
    eliminated), with first-order upwind convection along x when conv > 0."""
    n = m ** dim
    idx = torch.arange(n, device="cuda", dtype=torch.int64)
    entries = []   # (offset, valid, value), columns ascending
    for axis in reversed(range(dim)):
        entries.append((-(m ** axis), (idx // m ** axis) % m > 0, -1.0 - (conv if axis == 0 else 0.0)))
    entries.append((0, None, 2.0 * dim + conv))
    for axis in range(dim):
        entries.append((m ** axis, (idx // m ** axis) % m < m - 1, -1.0))
    counts = torch.zeros(n, device="cuda", dtype=torch.int64)
    for _, ok, _ in entries:
        counts += 1 if ok is None else ok
    rowptr = torch.zeros(n + 1, device="cuda", dtype=torch.int64)
    torch.cumsum(counts, 0, out=rowptr[1:])
    nnz = int(rowptr[-1])
    col = torch.empty(nnz, device="cuda", dtype=torch.int32)
    val = torch.empty(nnz, device="cuda", dtype=torch.float64)
    pos = rowptr[:-1].clone()
    for off, ok, v in entries:
        rows = idx if ok is None else idx[ok]
        p = pos if ok is None else pos[ok]
        col[p] = (rows + off).to(torch.int32)
        val[p] = v
        if ok is None:
            pos += 1
        else:
            pos += ok
    return rowptr.to(torch.int32), col, val


def _injection_csr(mc):
    mf = 2 * mc + 1
    k = torch.arange(mc * mc, device="cuda", dtype=torch.int64)
    col = (2 * (k // mc) + 1) * mf + 2 * (k % mc) + 1
    one = torch.ones(mc * mc, device="cuda", dtype=torch.float64)
    return torch.arange(mc * mc + 1, device="cuda", dtype=torch.int32), col.to(torch.int32), one


def _bilinear_csr(mc):
    mf = 2 * mc + 1
    k = torch.arange(mf * mf, device="cuda", dtype=torch.int64)

    def axis(i):
        odd = i % 2 == 1
        one, half = (torch.full(i.shape, v, device="cuda", dtype=torch.float64) for v in (1.0, 0.5))
        return ((torch.where(odd, (i - 1) // 2, i // 2 - 1), torch.where(odd, one, half)),
                (torch.where(odd, torch.full_like(i, -1), i // 2), torch.where(odd, one * 0, half)))

    cols, vals = [], []
    for cj, wj in axis(k // mf):
        for ci, wi in axis(k % mf):
            ok = (cj >= 0) & (cj < mc) & (ci >= 0) & (ci < mc) & (wj > 0) & (wi > 0)
            cols.append(torch.where(ok, cj * mc + ci, torch.full_like(k, -1)))
            vals.append(wj * wi)
    col, val = torch.stack(cols, 1), torch.stack(vals, 1)
    keep = col >= 0
    rowptr = torch.zeros(mf * mf + 1, device="cuda", dtype=torch.int64)
    torch.cumsum(keep.sum(1), 0, out=rowptr[1:])
    return rowptr.to(torch.int32), col[keep].to(torch.int32), val[keep]


def _sides(case):
    c, lo, hi = case["count"], case["lo"], case["hi"]
    return [lo + (hi - lo) * ((7 * i) % c) // max(1, c - 1) for i in range(c)]


# ---------------------------------------------------------------- stores
DT = {torch.float64: "f64", torch.float32: "f32", torch.int32: "i32"}


def _wrap(s, t):
    """A store over a tensor of the program's own."""
    s.setdefault("tensors", []).append(t)
    return s["ctx"].store_wrap(t.data_ptr(), list(t.shape), DT[t.dtype])


class _Device:
    def __init__(self, ctx, store, shape, dtype):
        self.ctx = ctx
        self.__cuda_array_interface__ = {"shape": tuple(shape), "typestr": "<f8" if dtype == "f64" else "<f4",
                                         "data": (ctx.store_device_ptr(store), False), "strides": None, "version": 3}


def _view(ctx, store, shape, dtype="f64"):
    """A tensor over a store's memory."""
    return torch.as_tensor(_Device(ctx, store, shape, dtype), device="cuda")


def _settle(c, step):
    """One pass, its kernels compiled, one more so that they are loaded."""
    step()
    c.sync()
    dfx.jit_wait()
    step()
    c.sync()
    dfx.jit_wait()


_STREAM = []


def _context(**kw):
    """A context on the program's one stream: its solves run one after another."""
    if not _STREAM:
        _STREAM.append(torch.cuda.Stream())
    return dfx.Context(device=0, stream=_STREAM[0].cuda_stream, **kw)


# ---------------------------------------------------------------- prepare
def prepare(case, seed):
    s = {"case": case}
    kind = case["kind"]
    if kind == "serve":
        return _prepare_serve(s, seed)
    if kind == "batch":
        return _prepare_batch(s, seed)
    window = 64 if kind == "price" else 16
    s["ctx"] = c = _context(window_size=window, jit=case["jit"])
    if kind == "price":
        dt = TORCH[case["dtype"]]
        s["in"] = [_wrap(s, t) for t in _price_inputs(case, seed)]
        s["r"], s["sig"] = (_wrap(s, torch.tensor(v, device="cuda", dtype=dt)) for v in (RATE, VOL))
        torch.cuda.synchronize()
        s["rv"] = dfx.apps.bs_drift(c, s["r"], s["sig"], case["dtype"])
        s["out"] = None
        _settle(c, lambda: _price(s))
    elif kind == "sweep":
        grid = _sweep_input(case, seed)
        start = grid.clone()
        s["G"] = _wrap(s, grid)
        s["grid"] = grid
        torch.cuda.synchronize()
        s["jac"] = dfx.apps.Jacobi(c, s["G"], case["N"])
        _settle(c, lambda: run(s))
        grid.copy_(start)
    elif kind == "table":
        X, mu, sd, w = _table_inputs(case, seed)
        s["z"] = torch.zeros_like(X)
        s["h"] = [_wrap(s, t) for t in (X, mu, sd, w, s["z"])]
        torch.cuda.synchronize()
        s["full"] = c.part_tiling([case["rows"], case["cols"]])
        s["bycol"] = c.part_tiling([case["cols"]], proj=c.proj_drop(2, 0b10))
        s["byrow"] = c.part_tiling([case["rows"]], proj=c.proj_drop(2, 0b01))
        s["ss"] = c.store_create([], case["dtype"])
        _settle(c, lambda: _table(s))
    elif kind == "gmg":
        _prepare_gmg(s, seed)
    else:
        _prepare_krylov(s, seed)
    torch.cuda.synchronize()
    return s


def _price_inputs(case, seed):
    n, dt = case["n"], TORCH[case["dtype"]]
    return [_uniform(n, 10.0, 100.0, dt, seed, 0), _uniform(n, 10.0, 100.0, dt, seed, 1),
            _uniform(n, 0.25, 2.0, dt, seed, 2)]


def _sweep_input(case, seed):
    return _uniform((case["N"], case["N"]), 0.0, 1.0, torch.float64, seed, 0)


def _table_inputs(case, seed):
    r, k, dt = case["rows"], case["cols"], TORCH[case["dtype"]]
    return (_uniform((r, k), -2.0, 5.0, dt, seed, 0), _uniform(k, 1.0, 2.0, dt, seed, 1),
            _uniform(k, 0.5, 3.0, dt, seed, 2), _uniform(r, 0.0, 1.0, dt, seed, 3))


def _rhs(n, seed, k=0):
    return _uniform(n, -1.0, 1.0, torch.float64, seed, k)


def _record(s, solver):
    """One iteration recorded as a graph, as a program replays it."""
    c = s["ctx"]
    _settle(c, solver.iteration)
    s["graph"] = None
    if s["case"]["graph"]:
        c.graph_begin()
        solver.iteration()
        s["graph"] = c.graph_end()
        c.sync()


def _prepare_krylov(s, seed):
    case, c = s["case"], s["ctx"]
    m, dim = case["m"], case["dim"]
    n = m ** dim
    A = _stencil_csr(m, dim, 0.5 if case["kind"] == "bicgstab" else 0.0)
    h = [_wrap(s, t) for t in A]
    s["b"] = _wrap(s, _rhs(n, seed))
    torch.cuda.synchronize()
    s["solver"] = (dfx.apps.CG if case["kind"] == "cg" else dfx.apps.BiCGSTAB)(c, *h, s["b"], n)
    _record(s, s["solver"])
    g = s["solver"]
    names = ("x", "r", "p") if case["kind"] == "cg" else ("x", "r", "p", "v")
    s["views"] = [_view(c, getattr(g, k), [n]) for k in names]
    s["views"].append(_view(c, g.rho if case["kind"] == "cg" else g.rr, []))
    _settle(c, lambda: run(s))   # the restart's passes, and an eager loop's own windows


def _prepare_gmg(s, seed):
    case, c = s["case"], s["ctx"]
    m, levels, sizes = case["m"], [], []
    for l in range(case["levels"]):
        rp, col, val = _stencil_csr(m, 2)
        sizes.append(m * m)
        A = tuple(_wrap(s, t) for t in (rp, col, val * 0.25 ** l))
        R = P = None
        if l < case["levels"] - 1:
            m = (m - 1) // 2
            R = tuple(_wrap(s, t) for t in _injection_csr(m))
            P = tuple(_wrap(s, t) for t in _bilinear_csr(m))
        levels.append((A, 4.0 * 0.25 ** l, R, P))
    s["b"] = _wrap(s, _rhs(sizes[0], seed))
    torch.cuda.synchronize()
    g = s["solver"] = dfx.apps.GMG(c, levels, sizes, s["b"])
    # the first direction and its product with the residual, kept so that the
    # solve can start again
    T, N = c.part_tiling([sizes[0]]), c.part_none()
    s["T"], s["N"] = T, N
    s["p0"], s["rho0"] = c.store_create([sizes[0]], "f64"), c.store_create([], "f64")
    c.submit("copy", [1], [(g.p, T, "R"), (s["p0"], T, "W")])
    c.submit("copy", [], [(g.rho, N, "R"), (s["rho0"], N, "W")])
    c.sync()
    _record(s, g)
    s["views"] = [_view(c, h, [sizes[0]]) for h in (g.x, g.r, g.z, g.p)] + [_view(c, h, []) for h in (g.rho, g.rr)]
    _settle(c, lambda: run(s))   # the restart's passes, and an eager loop's own windows


def _prepare_batch(s, seed):
    s["batch"] = b = dfx.Batch(device=0)
    s["ctxs"], s["views"] = [], []
    for i, m in enumerate(_sides(s["case"])):
        c = _context(window_size=16)
        t = list(_stencil_csr(m, 2)) + [_rhs(m * m, seed, i)]
        torch.cuda.synchronize()
        h = [c.store_wrap(v.data_ptr(), list(v.shape), DT[v.dtype]) for v in t]
        none, rho0 = c.part_none(), c.store_create([], "f64")
        # an untimed solve's first passes give every store its memory
        cg = dfx.apps.CG(c, *h, m * m)
        c.submit("copy", [], [(cg.rho, none, "R"), (rho0, none, "W")])
        cg.iteration()
        c.sync()
        b.record_begin(c)
        _restart_cg(c, cg, h[3])
        c.submit("copy", [], [(cg.rho, none, "R"), (rho0, none, "W")])
        b.loop_begin(c)
        cg.iteration()
        b.record_end(c, max_iter=20000, conv_a=cg.rho, conv_b=rho0, tol=1e-16)
        s["ctxs"].append((c, cg, t))
        s["views"].append(_view(c, cg.x, [m * m]))
    return s


def _prepare_serve(s, seed):
    s["ctx"] = c = _context()
    mats = {m: [t.cpu().numpy() for t in _stencil_csr(m, 2)] for m in set(_sides(s["case"]))}
    s["req"] = [(mats[m], _rhs(m * m, seed, i).cpu().numpy()) for i, m in enumerate(_sides(s["case"]))]
    c.serve_start(hbm_budget=4 << 30, max_slots=64, tol=1e-8, max_iter=20000)
    return s


# ---------------------------------------------------------------- run
def _price(s):
    c, case = s["ctx"], s["case"]
    if s["out"]:
        c.store_release(s["out"][0])
        c.store_release(s["out"][1])
    s["out"] = dfx.apps.black_scholes(c, *s["in"], s["r"], s["sig"], s["rv"], case["n"], case["dtype"])
    c.flush()


def _table(s):
    c, case = s["ctx"], s["case"]
    X, mu, sd, w, z = s["h"]
    F, by, br, d, dt = s["full"], s["bycol"], s["byrow"], [1, 1], case["dtype"]
    t1, t2 = (c.store_create([case["rows"], case["cols"]], dt) for _ in range(2))
    c.submit("sub", d, [(X, F, "R"), (mu, by, "R"), (t1, F, "W")])
    c.submit("div", d, [(t1, F, "R"), (sd, by, "R"), (t2, F, "W")])
    c.submit("mul", d, [(t2, F, "R"), (w, br, "R"), (z, F, "W")])
    c.store_release(t1)
    c.store_release(t2)
    c.submit("sumsq", d, [(z, F, "R"), (s["ss"], c.part_none(), "Rd")], (1,))
    c.flush()


def _restart_cg(c, g, b):
    T, N, d = g.tile, g.none, g.d
    c.submit("fill", d, [(g.x, T, "W")], (0.0,))
    c.submit("copy", d, [(b, T, "R"), (g.r, T, "W")])
    c.submit("copy", d, [(g.r, T, "R"), (g.p, T, "W")])
    c.submit("dot", d, [(g.r, T, "R"), (g.r, T, "R"), (g.rho, N, "Rd")], (1,))


def _restart_bicgstab(c, g, b):
    T, N, d = g.tile, g.none, g.d
    c.submit("fill", d, [(g.x, T, "W")], (0.0,))
    c.submit("copy", d, [(b, T, "R"), (g.r, T, "W")])
    c.submit("copy", d, [(b, T, "R"), (g.rhat, T, "W")])
    c.submit("fill", d, [(g.p, T, "W")], (0.0,))
    c.submit("fill", d, [(g.v, T, "W")], (0.0,))
    for k in (g.rho, g.alpha, g.omega):
        c.submit("fill", [], [(k, N, "W")], (1.0,))
    c.submit("dot", d, [(g.r, T, "R"), (g.r, T, "R"), (g.rr, N, "Rd")], (1,))
    c.submit("dot", d, [(g.rhat, T, "R"), (g.r, T, "R"), (g.rho_new, N, "Rd")], (1,))


def _restart_gmg(s):
    c, g, T, N = s["ctx"], s["solver"], s["T"], s["N"]
    c.submit("fill", [1], [(g.x, T, "W")], (0.0,))
    c.submit("copy", [1], [(s["b"], T, "R"), (g.r, T, "W")])
    c.submit("copy", [1], [(s["p0"], T, "R"), (g.p, T, "W")])
    c.submit("copy", [], [(s["rho0"], N, "R"), (g.rho, N, "W")])


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "price":
        _price(s)
        return [_view(s["ctx"], h, [case["n"]], case["dtype"]) for h in s["out"]]
    if kind == "sweep":
        for _ in range(case["sweeps"]):
            res = s["jac"].sweep()
        s["ctx"].flush()
        return [s["grid"], _view(s["ctx"], res, [])]
    if kind == "table":
        _table(s)
        return [s["z"], _view(s["ctx"], s["ss"], [], case["dtype"])]
    if kind == "batch":
        s["batch"].run()
        s["batch"].wait()
        its = np.array([s["batch"].stream_info(i)[0] for i in range(case["count"])])
        return s["views"] + [its]
    if kind == "serve":
        return _serve(s)
    c, g = s["ctx"], s["solver"]
    if kind == "cg":
        _restart_cg(c, g, s["b"])
    elif kind == "bicgstab":
        _restart_bicgstab(c, g, s["b"])
    else:
        _restart_gmg(s)
    c.flush()
    for _ in range(case["iters"]):
        if s["graph"] is not None:
            c.graph_launch(s["graph"])
        else:
            g.iteration()
    c.flush()
    return s["views"]


def _serve(s):
    c = s["ctx"]
    tickets = [c.serve_submit(*mat, b) for mat, b in s["req"]]
    out, its = [], []
    for t, (_, b) in zip(tickets, s["req"]):
        res = c.serve_wait(t)
        its.append((res["status"], res["iterations"]))
        out.append(c.serve_read_x(t, b.size))
        c.serve_release(t)
    return out + [np.array(its)]


# ---------------------------------------------------------------- work
def work(case):
    kind = case["kind"]
    if kind == "price":
        n, e = case["n"], 8 if case["dtype"] == "f64" else 4
        return {"bytes": 5 * n * e, "flops": 28 * n}
    if kind == "sweep":
        pts = (case["N"] - 2) ** 2
        # grid in, work out; work in, grid out; six adds and multiplies, three for the residual
        return {"bytes": 32 * pts * case["sweeps"], "flops": 8 * pts * case["sweeps"]}
    if kind == "table":
        n, e = case["rows"] * case["cols"], 8 if case["dtype"] == "f64" else 4
        return {"bytes": (2 * n + 2 * case["cols"] + case["rows"]) * e, "flops": 5 * n}
    if kind in ("cg", "bicgstab"):
        n, per = case["m"] ** case["dim"], 2 * case["dim"] + 1
        mat = n * (12 * per + 4)
        # CG: matrix, p in, q out; x, r read and written, p, q in; p, r in, p out
        # BiCGSTAB: twice the matrix; p, r, v in, p out; v and t products;
        # r, v in, s out; x in and out, p, s, t, rhat in, r out
        vec = (16 + 48 + 24) if kind == "cg" else (32 + 24 + 24 + 24 + 56)
        return {"bytes": (mat * (1 if kind == "cg" else 2) + vec * n) * case["iters"],
                "flops": (2 * per + 10) * n * case["iters"] * (1 if kind == "cg" else 2)}
    if kind == "gmg":
        total, n = 0, case["m"] ** 2
        for l in range(case["levels"]):
            k = (((case["m"] + 1) >> l) - 1) ** 2
            last = l == case["levels"] - 1
            # per smoothing or residual: matrix, x and b in, r out, x in and out
            total += (8 if last else 5) * k * (64 + 40)
            if not last:
                total += k * (4 + 12 * 2.25 + 24)   # prolongation and correction
        return {"bytes": (total + n * (64 + 16 + 48 + 16 + 24)) * case["iters"], "flops": total / 6 * case["iters"]}
    # independent solves: about 2.9 iterations per unit of side at tol 1e-8
    rows = sum(2.9 * m * m * m for m in _sides(case))
    return {"bytes": rows * (64 + 16 + 48 + 24), "flops": rows * 20}


# ---------------------------------------------------------------- exact
def _apply(x, m, dim, conv=0.0):
    """The stencil matrix applied to a vector over the m^dim grid."""
    u = x.reshape([m] * dim)
    y = (2.0 * dim + conv) * u
    for axis in range(dim):   # tensor axis dim - 1 is x
        k = u.shape[axis]
        lo, hi = u.narrow(axis, 0, k - 1), u.narrow(axis, 1, k - 1)
        y.narrow(axis, 1, k - 1).sub_(lo, alpha=1.0 + (conv if axis == dim - 1 else 0.0))
        y.narrow(axis, 0, k - 1).sub_(hi)
    return y.reshape(-1)


def _cg(b, m, dim, iters, tol=None):
    x, r, p = torch.zeros_like(b), b.clone(), b.clone()
    rho = torch.dot(r, r)
    stop = None if tol is None else float(rho) * tol * tol
    for k in range(iters):
        q = _apply(p, m, dim)
        alpha = rho / torch.dot(p, q)
        x = x + alpha * p
        r = r - alpha * q
        new = torch.dot(r, r)
        p = p * (new / rho) + r
        rho = new
        if stop is not None and float(rho) <= stop:
            break
    return x, r, p, rho


def _vcycle(b, m, l, levels):
    scale, w = 0.25 ** l, (2.0 / 3.0) / (4.0 * 0.25 ** l)
    x = torch.zeros_like(b)
    res = lambda: b - scale * _apply(x, m, 2)
    if l == levels - 1:
        for _ in range(8):
            x = x + w * res()
        return x
    for _ in range(2):
        x = x + w * res()
    mc = (m - 1) // 2
    e = _vcycle(res().reshape(m, m)[1::2, 1::2].reshape(-1).contiguous(), mc, l + 1, levels).reshape(mc, mc)
    f = torch.zeros(m + 2, m + 2, device=b.device, dtype=b.dtype)   # fine grid with its zero boundary
    f[2:-2:2, 2:-2:2] = e
    f[1::2, :] = 0.5 * (f[0:-1:2, :] + f[2::2, :])
    f[:, 1::2] = 0.5 * (f[:, 0:-1:2] + f[:, 2::2])
    x = x + f[1:-1, 1:-1].reshape(-1)
    for _ in range(2):
        x = x + w * res()
    return x


def exact(case, seed):
    kind = case["kind"]
    if kind == "price":
        S, K, T = (t.double() for t in _price_inputs(case, seed))
        r, sig = (float(torch.tensor(v, dtype=TORCH[case["dtype"]])) for v in (RATE, VOL))
        vs = sig * torch.sqrt(T)
        d1 = (torch.log(S / K) + (r + 0.5 * sig * sig) * T) / vs
        N1 = 0.5 * torch.erfc(-d1 * math.sqrt(0.5))
        N2 = 0.5 * torch.erfc(-(d1 - vs) * math.sqrt(0.5))
        Kd = K * torch.exp(-r * T)
        return [S * N1 - Kd * N2, Kd * (1.0 - N2) - S * (1.0 - N1)]
    if kind == "sweep":
        g = _sweep_input(case, seed)
        for _ in range(case["sweeps"]):
            c = g[1:-1, 1:-1]
            work_ = 0.2 * (c + g[:-2, 1:-1] + g[1:-1, 2:] + g[1:-1, :-2] + g[2:, 1:-1])
            res = (work_ - c).square().sum().sqrt()
            g[1:-1, 1:-1] = work_
        return [g, res]
    if kind == "table":
        X, mu, sd, w = (t.double() for t in _table_inputs(case, seed))
        z = (X - mu) / sd * w[:, None]
        return [z, z.square().sum()]
    if kind == "cg":
        return list(_cg(_rhs(case["m"] ** case["dim"], seed), case["m"], case["dim"], case["iters"]))
    if kind == "bicgstab":
        m, dim = case["m"], case["dim"]
        b = _rhs(m ** dim, seed)
        x, p, v, r = torch.zeros_like(b), torch.zeros_like(b), torch.zeros_like(b), b.clone()
        rho = alpha = omega = torch.ones((), device="cuda", dtype=torch.float64)
        for _ in range(case["iters"]):
            new = torch.dot(b, r)
            p = (p - omega * v) * ((new / rho) * (alpha / omega)) + r
            rho = new
            v = _apply(p, m, dim, 0.5)
            alpha = rho / torch.dot(b, v)
            t_ = r - alpha * v
            t = _apply(t_, m, dim, 0.5)
            omega = torch.dot(t, t_) / torch.dot(t, t)
            x = x + alpha * p + omega * t_
            r = t_ - omega * t
        return [x, r, p, v, torch.dot(r, r)]
    if kind == "gmg":
        m, lev = case["m"], case["levels"]
        b = _rhs(m * m, seed)
        x, r = torch.zeros_like(b), b.clone()
        z = _vcycle(r, m, 0, lev)
        p, rho = z.clone(), torch.dot(r, z)
        for _ in range(case["iters"]):
            q = _apply(p, m, 2)
            alpha = rho / torch.dot(p, q)
            x = x + alpha * p
            r = r - alpha * q
            rr = torch.dot(r, r)
            z = _vcycle(r, m, 0, lev)
            new = torch.dot(r, z)
            p = p * (new / rho) + z
            rho = new
        return [x, r, z, p, rho, rr]
    # batch and serve: every solve's x; iteration counts have no exact value
    return [_cg(_rhs(m * m, seed, i), m, 2, 20000, 1e-8)[0] for i, m in enumerate(_sides(case))] + [None]
