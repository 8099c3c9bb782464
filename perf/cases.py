"""The work that users of this library have it do, as cases to be timed.

A case is a dict of plain values; `prepare` makes what a program holds before
the call (inputs on the GPU and the solver handle it keeps), `run` takes one
pass through the public entry points and returns the whole outputs, `work`
states what a pass cannot do without and `exact` gives the same outputs in
64-bit torch arithmetic.

Kinds of pass:
  solve     set source, set state, sweeps with a residual every `every`
            sweeps, read the state back (Solver; 2D and 3D, FP32 and FP64,
            Poisson and Laplace; `explicit`: halos exchanged before every sweep)
  noalloc   the same solve through the entry point without a workspace
  monitor   sweep / residual-to-host in a loop, as a program does that decides
            on the host when to stop
  batch     grids of uneven sizes solved together with the stop rule
  gradient  differentiable sweeps: forward, then the gradients of a loss
"""
import ctypes
import math
import random

import torch

import paper_2303_02543_amd as jb
from paper_2303_02543_amd.autograd import jacobi_k

DTYPES = {"f32": torch.float32, "f64": torch.float64}


def _valid_blocks(n, b, dtype, axis):
    """The largest block count <= b the library accepts for n nodes on an axis
    (x extents are rounded up to 32 bytes; the last block must not be empty)."""
    b = max(1, min(b, n))
    while b > 1:
        e = -(-n // b)
        if axis == 0:
            g = 32 // (torch.finfo(DTYPES[dtype]).bits // 8)
            e = -(-e // g) * g
        if (b - 1) * e < n:
            break
        b -= 1
    return b


def _grid(case):
    return tuple(case[a] for a in ("nx", "ny", "nz") if a in case)


def _blocks(case):
    return tuple(case[a] for a in ("bx", "by", "bz") if a in case)


def listed():
    return [
        # the smallest call: one short solve of a small grid in a serving
        # loop; bound by launches (sizes of the repository's smoke run)
        {"name": "noalloc_130_f32", "kind": "noalloc", "nx": 130, "ny": 130, "bx": 2, "by": 3,
         "dtype": "f32", "source": True, "sweeps": 24, "every": 8},
        # the repository's FP64 Laplace case: a small grid in double precision
        {"name": "laplace_256_f64", "kind": "solve", "nx": 256, "ny": 256, "bx": 2, "by": 2,
         "dtype": "f64", "source": False, "sweeps": 100, "every": 10},
        # a small 3D domain, a few blocks per axis
        {"name": "poisson3d_96_f32", "kind": "solve", "nx": 96, "ny": 96, "nz": 96, "bx": 2,
         "by": 2, "bz": 2, "dtype": "f32", "source": True, "sweeps": 40, "every": 10},
        # an ordinary ragged grid, the host watching the residual
        {"name": "monitor_1000x777_f32", "kind": "monitor", "nx": 1000, "ny": 777, "bx": 4,
         "by": 3, "dtype": "f32", "source": True, "sweeps": 100, "every": 25},
        # the benchmark's workload: large 2D FP32 Poisson
        {"name": "poisson_8192_f32", "kind": "solve", "nx": 8192, "ny": 8192, "bx": 16,
         "by": 16, "dtype": "f32", "source": True, "sweeps": 1000, "every": 50},
        # a middling ragged 2D grid in double precision
        {"name": "poisson_2500x1701_f64", "kind": "solve", "nx": 2500, "ny": 1701, "bx": 5,
         "by": 4, "dtype": "f64", "source": True, "sweeps": 200, "every": 50},
        # the paper's step order (halo exchange, then a block-local update)
        {"name": "explicit_4096_f32", "kind": "solve", "nx": 4096, "ny": 4096, "bx": 16,
         "by": 16, "dtype": "f32", "source": True, "sweeps": 100, "every": 50, "explicit": True},
        # the benchmark's 3D workload
        {"name": "poisson3d_512_f32", "kind": "solve", "nx": 512, "ny": 512, "nz": 512, "bx": 8,
         "by": 8, "bz": 8, "dtype": "f32", "source": True, "sweeps": 200, "every": 20},
        # a ragged 3D domain in double precision
        {"name": "poisson3d_350x301x260_f64", "kind": "solve", "nx": 350, "ny": 301, "nz": 260,
         "bx": 5, "by": 5, "bz": 4, "dtype": "f64", "source": True, "sweeps": 100, "every": 20},
        # grids of uneven sizes solved together, as the batched benchmark draws them
        {"name": "batch_12_f32", "kind": "batch", "count": 12, "lo": 257, "hi": 2049,
         "sizes_seed": 4, "block": 512, "dtype": "f32", "sweeps": 500, "every": 50, "tol": 1e-6},
        # the gradient workload: forward and backward through many sweeps
        {"name": "gradient_4096_f32", "kind": "gradient", "nx": 4096, "ny": 4096, "bx": 8,
         "by": 8, "dtype": "f32", "source": True, "sweeps": 500, "chunk": 50},
        # a small gradient in double precision, as inside an optimisation loop
        {"name": "gradient_300x201_f64", "kind": "gradient", "nx": 300, "ny": 201, "bx": 2,
         "by": 2, "dtype": "f64", "source": True, "sweeps": 60, "chunk": 20},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["noalloc", "solve2", "solve2", "solve3", "solve3", "monitor", "explicit",
                       "batch", "gradient"])
    dtype = rng.choice(["f32", "f64"])
    c = {"dtype": dtype}
    if kind == "batch":
        hi = _log_int(rng, 300, 2100)
        c.update(kind="batch", count=rng.randint(3, 14), lo=rng.randint(20, 257), hi=hi,
                 sizes_seed=rng.randint(0, 10 ** 6), block=rng.choice([128, 256, 512]),
                 sweeps=_log_int(rng, 40, 600), every=rng.choice([10, 25, 50]), tol=1e-6)
        return c
    if kind == "solve3":
        n = _log_int(rng, 40, 420)
        axes = {a: max(9, int(n * rng.uniform(0.7, 1.25))) for a in ("nx", "ny", "nz")}
        side = rng.choice([32, 48, 64])
    else:
        top = {"noalloc": 1400 if dtype == "f32" else 900, "solve2": 6000, "monitor": 3000,
               "explicit": 5000, "gradient": 3000}[kind]
        n = _log_int(rng, 100, top)
        axes = {a: max(9, int(n * rng.uniform(0.7, 1.25))) for a in ("nx", "ny")}
        side = rng.choice([64, 128, 256, 512])
    c.update(axes)
    for k, (a, b) in enumerate((("nx", "bx"), ("ny", "by"), ("nz", "bz"))):
        if a in c:
            c[b] = _valid_blocks(c[a], -(-c[a] // side), dtype, k)
    c["source"] = kind in ("gradient",) or rng.random() < 0.75
    c["sweeps"] = _log_int(rng, 20, 200 if kind in ("solve3", "explicit", "gradient") else 400)
    if kind == "gradient":
        c["chunk"] = max(1, c["sweeps"] // rng.randint(1, 8))
    else:
        c["every"] = rng.choice([10, 20, 25, 50])
    if kind == "explicit":
        c["explicit"] = True
    c["kind"] = {"solve2": "solve", "solve3": "solve", "explicit": "solve"}.get(kind, kind)
    return c


# ------------------------------------------------------------------ inputs
def _gen(seed, k=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * int(seed) + k)
    return g


def _gaussians(shape, seed, k):
    """Sum of 16 Gaussians over the unit square / cube (centres U[0,1), sigma
    U[0.01, 0.05], amplitudes N(0,1)), in FP64 on the GPU."""
    r = random.Random(1000003 * int(seed) + k)
    nd = len(shape)
    fac = [[] for _ in range(nd)]
    for _ in range(16):
        centre = [r.random() for _ in range(nd)]
        s = r.uniform(0.01, 0.05)
        amp = r.gauss(0.0, 1.0)
        for a, n in enumerate(shape):
            x = torch.arange(1, n + 1, dtype=torch.float64, device="cuda") / (n + 1)
            e = torch.exp(-((x - centre[a]) ** 2) / (2 * s * s))
            fac[a].append(e * amp if a == 0 else e)
    m = [torch.stack(v) for v in fac]
    if nd == 2:
        return m[0].t().contiguous() @ m[1]
    rest = (m[1][:, :, None] * m[2][:, None, :]).reshape(16, -1)
    return (m[0].t().contiguous() @ rest).reshape(shape)


def _uniform(shape, seed, k, lo, hi):
    return torch.rand(shape, generator=_gen(seed, k), dtype=torch.float64, device="cuda") * \
        (hi - lo) + lo


def _inputs(case, seed):
    """(U0 full state, f interior source or None, h2) of a single grid, in the
    case's dtype."""
    dt = DTYPES[case["dtype"]]
    shape = tuple(reversed(_grid(case)))
    full = tuple(n + 2 for n in shape)
    h2 = 1.0 / (max(shape) + 1) ** 2
    f = None
    if len(shape) == 3:
        U0 = torch.zeros(full, dtype=dt, device="cuda")
        if case["source"]:
            f = _uniform(shape, seed, 1, -1.0, 1.0).to(dt)
        else:
            U0[-1] = 1.0
            U0[1:-1, 1:-1, 1:-1] = _uniform(shape, seed, 2, 0.0, 1.0)
    elif case["source"]:
        # Gaussian sources; ring values for the gradient, a zero ring otherwise
        f = _gaussians(shape, seed, 1).to(dt)
        U0 = torch.zeros(full, dtype=dt, device="cuda")
        if case["kind"] == "gradient":
            ring = _uniform(full, seed, 3, 0.0, 1.0)
            ring[1:-1, 1:-1] = 0.0
            U0 = ring.to(dt)
    else:
        # Laplace: one edge held at 1, a random start inside
        U0 = torch.zeros(full, dtype=dt, device="cuda")
        U0[-1, 1:-1] = 1.0
        U0[1:-1, 1:-1] = _uniform(shape, seed, 2, 0.0, 1.0)
    return U0, f, h2


def _batch_sizes(case):
    r = random.Random(case["sizes_seed"])
    lo, hi = min(case["lo"], case["hi"]), max(case["lo"], case["hi"])
    return [(r.randint(lo, hi), r.randint(lo, hi)) for _ in range(case["count"])]


def _batch_inputs(case, seed):
    dt = DTYPES[case["dtype"]]
    grids, us, fs, h2s = _batch_sizes(case), [], [], []
    for k, (nx, ny) in enumerate(grids):
        us.append(torch.zeros((ny + 2, nx + 2), dtype=dt, device="cuda"))
        fs.append(_gaussians((ny, nx), seed, 10 + k).to(dt))
        h2s.append(1.0 / (max(nx, ny) + 1) ** 2)
    return grids, us, fs, h2s


def _target(case, seed):
    shape = tuple(n + 2 for n in reversed(_grid(case)))
    return _gaussians(shape, seed, 5).to(DTYPES[case["dtype"]])


# ------------------------------------------------------------- the GPU path
def prepare(case, seed):
    dt = DTYPES[case["dtype"]]
    if case["kind"] == "batch":
        grids, us, fs, h2s = _batch_inputs(case, seed)
        return {"case": case, "b": jb.Batch(grids, dt, block=case["block"],
                                             device="cuda:0"), "us": us, "fs": fs,
                "h2s": h2s}
    U0, f, h2 = _inputs(case, seed)
    st = {"case": case, "u0": U0, "f": f, "h2": h2}
    if case["kind"] == "noalloc":
        st["out"] = torch.empty_like(U0)
        st["res"] = torch.empty(jb.residual_count(case["sweeps"], case["every"]),
                                dtype=torch.float64, device="cuda")
        return st
    st["s"] = jb.Solver(_grid(case), _blocks(case), dt)
    if case.get("explicit"):
        st["s"].set_tuning(1, 0, jb.JACOBI_FLAG_EXPLICIT_HALO)
    if case["kind"] == "gradient":
        st["f"] = f.requires_grad_(True)
        st["u0"] = U0.requires_grad_(True)
        st["target"] = _target(case, seed)
    return st


def _ptr(t):
    return None if t is None else ctypes.c_void_p(t.data_ptr())


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "noalloc":
        stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
        jb.jacobi_solve_noalloc(len(_grid(case)), _grid(case), _blocks(case),
                                jb.dtype_code(DTYPES[case["dtype"]]), _ptr(st["u0"]),
                                _ptr(st["f"]), st["h2"], case["sweeps"], case["every"],
                                _ptr(st["out"]), _ptr(st["res"]), stream)
        return {"u": st["out"], "res": st["res"]}
    if kind == "batch":
        b = st["b"]
        for i in range(b.count):
            b.set_grid(i, st["us"][i], st["fs"][i], st["h2s"][i])
        sweeps, rel, status = b.solve(case["tol"], case["sweeps"], case["every"])
        return {"u": [b.get_grid(i) for i in range(b.count)], "sweeps": sweeps, "rel": rel,
                "status": status}
    if kind == "gradient":
        u = jacobi_k(st["f"], st["u0"], st["s"], case["sweeps"], st["h2"], case["chunk"])
        df, du0 = torch.autograd.grad(u, (st["f"], st["u0"]), u.detach() - st["target"])
        return {"u": u.detach(), "df": df, "du0": du0}
    s = st["s"]
    s.set_source(st["f"], st["h2"])
    s.set_state(st["u0"])
    if kind == "monitor":
        seen = []
        left = case["sweeps"]
        while left > 0:
            n = min(case["every"], left)
            s.sweep(n)
            seen.append(s.residual())
            left -= n
        return {"u": s.get_state(), "res": seen}
    res = s.solve(case["sweeps"], case["every"])
    return {"u": s.get_state(), "res": res}


# ---------------------------------------------------------------- the work
def work(case):
    es = torch.finfo(DTYPES[case["dtype"]]).bits // 8
    if case["kind"] == "batch":
        cells = [nx * ny for nx, ny in _batch_sizes(case)]
        full = [(nx + 2) * (ny + 2) for nx, ny in _batch_sizes(case)]
        # with this tolerance and these sweeps every larger grid runs to the cap
        return {"bytes": es * (2 * sum(full) + sum(cells)),
                "flops": 5.0 * sum(cells) * case["sweeps"]}
    grid = _grid(case)
    cells = math.prod(grid)
    full = math.prod(n + 2 for n in grid)
    per = (7 if len(grid) == 3 else 5) - (0 if case["source"] else 1)
    nbytes = es * (2 * full + (cells if case["source"] else 0))
    flops = float(per) * cells * case["sweeps"]
    if case["kind"] == "gradient":
        # the target gradient in, dL/df and dL/dU0 out; the transposed sweep
        # (4) and the accumulation w * lam (2) per cell and sweep
        nbytes += es * (2 * full + cells)
        flops += 6.0 * cells * case["sweeps"]
    return {"bytes": nbytes, "flops": flops}


# ------------------------------------------------------- 64-bit plain torch
def _neighbours(U):
    if U.dim() == 2:
        return (U[1:-1, :-2] + U[1:-1, 2:]) + (U[:-2, 1:-1] + U[2:, 1:-1])
    return ((U[1:-1, 1:-1, :-2] + U[1:-1, 1:-1, 2:]) + (U[1:-1, :-2, 1:-1] + U[1:-1, 2:, 1:-1])) \
        + (U[:-2, 1:-1, 1:-1] + U[2:, 1:-1, 1:-1])


def _inside(U):
    return U[(slice(1, -1),) * U.dim()]


def _sweeps64(U, b, n):
    w = 1.0 / (2 * U.dim())
    for _ in range(n):
        s = _neighbours(U)
        if b is not None:
            s += b
        s *= w
        _inside(U).copy_(s)
    return U


def _residual64(U, b):
    r = _neighbours(U) - 2.0 * U.dim() * _inside(U)
    if b is not None:
        r += b
    return float(torch.linalg.vector_norm(r))


def exact(case, seed):
    with torch.no_grad():
        if case["kind"] == "batch":
            grids, us, fs, h2s = _batch_inputs(case, seed)
            out = {"u": [], "sweeps": [], "rel": [], "status": []}
            for u, f, h2 in zip(us, fs, h2s):
                U, b = u.double(), f.double() * h2
                r0, k, rel, status = _residual64(U, b), 0, 0.0, 1
                while r0 > 0.0:
                    step = min(case["every"], case["sweeps"] - k)
                    _sweeps64(U, b, step)
                    k += step
                    rel = _residual64(U, b) / r0
                    status = 1 if rel <= case["tol"] else 2
                    if status == 1 or k >= case["sweeps"]:
                        break
                out["u"].append(U)
                out["sweeps"].append(k)
                out["rel"].append(rel)
                out["status"].append(status)
            return out
        U0, f, h2 = _inputs(case, seed)
        U = U0.double()
        b = None if f is None else f.double() * h2
        if case["kind"] == "gradient":
            _sweeps64(U, b, case["sweeps"])
            d = U - _target(case, seed).double()
            lam = d.clone()
            lam[0], lam[-1], lam[:, 0], lam[:, -1] = 0.0, 0.0, 0.0, 0.0
            acc = torch.zeros_like(b)
            for _ in range(case["sweeps"]):
                acc += 0.25 * _inside(lam)
                _sweeps64(lam, None, 1)
            du0 = d.clone()
            du0[1:-1, 1:-1] = _inside(lam)
            du0[0, 1:-1] += acc[0]
            du0[-1, 1:-1] += acc[-1]
            du0[1:-1, 0] += acc[:, 0]
            du0[1:-1, -1] += acc[:, -1]
            return {"u": U, "df": h2 * acc, "du0": du0}
        res = [] if case["kind"] == "monitor" else [_residual64(U, b)]
        k = 0
        while k < case["sweeps"]:
            step = min(case["every"], case["sweeps"] - k)
            _sweeps64(U, b, step)
            k += step
            res.append(_residual64(U, b))
        if case["kind"] != "monitor":
            res = torch.tensor(res, dtype=torch.float64)
        return {"u": U, "res": res}
