"""Cases of the SpMV and Krylov paths: what they run and what one pass costs.

Each case is a plain dict; ``prepare`` makes a program's state for it on the
GPU (inputs from the seed, matrix handles, hierarchies, a server), ``run`` is
one pass through the public entry points, ``work`` the bytes and operations a
pass cannot do without, and ``exact`` the same outputs in plain 64-bit torch.

Kinds:
  solve     Jacobi-PCG on a handle the program keeps, a new right-hand side
  spmv      one sparse matrix-vector product with scattered columns
  multi     k right-hand sides sharing every product
  smooth    Chebyshev-Jacobi smoothing steps
  mg        multigrid-preconditioned CG on a hierarchy the program keeps
  assemble  a new matrix each pass: handle, hierarchy, solve, release
  parts     a program's own Krylov step from the library's vector kernels
  serve     a burst of differently sized systems through the batching server
"""

from __future__ import annotations

import math

import numpy as np
import torch

import spkgen
from paper_2011_00715_amd import spk

DEV = "cuda"


def listed():
    return [
        # the smallest solve that programs bring: 64 x 64 five-point Poisson;
        # every launch and every reduction shows
        {"name": "solve_2d_64", "kind": "solve", "grid": "64x64", "stencil": "axis", "precision": "fp64"},
        # an ordinary 3D pressure solve on a grid of no particular size
        {"name": "solve_3d_ragged", "kind": "solve", "grid": "61x47x53", "stencil": "axis", "precision": "fp64"},
        # the seven-point 128^3 benchmark system, both precisions
        {"name": "solve_3d_128", "kind": "solve", "grid": "128x128x128", "stencil": "axis", "precision": "fp64"},
        {"name": "solve_3d_128_mixed", "kind": "solve", "grid": "128x128x128", "stencil": "axis",
         "precision": "mixed"},
        # the 27-point variable-coefficient diffusion benchmark, larger than any cache
        {"name": "solve_27pt_160", "kind": "solve", "grid": "160x160x160", "stencil": "box", "precision": "fp64"},
        # the power-law benchmark product: long and short rows, columns everywhere
        {"name": "spmv_powerlaw_4m", "kind": "spmv", "n": 4000000, "precision": "fp64"},
        # eight right-hand sides of one matrix
        {"name": "multi_8_128", "kind": "multi", "grid": "128x128x128", "k": 8},
        # the smoother alone, as a program's own multigrid calls it
        {"name": "smooth_2_128", "kind": "smooth", "grid": "128x128x128", "steps": 2, "residual": False},
        # multigrid-preconditioned solve, the fastest way to solve the 128^3 system
        {"name": "mg_128", "kind": "mg", "grid": "128x128x128", "precision": "fp64", "cycle": 1},
        # a time or Newton step whose matrix is new: assembly hands over CSR,
        # the library sets up the hierarchy, solves once and lets go
        {"name": "assemble_mg_ragged", "kind": "assemble", "grid": "97x64x81", "mg": True},
        # the building blocks, for a Krylov method the program writes itself
        {"name": "parts_3d", "kind": "parts", "grid": "127x131x113"},
        # a burst of requests of the served stream's mix (half 2D, half 3D)
        {"name": "serve_16", "kind": "serve", "count": 16, "mix": 1, "side2d": 256, "side3d": 80},
    ]


def _side(rng, lo, hi):
    """An extent between lo and hi, spread over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _grid(rng, dim, lo, hi):
    s = _side(rng, lo, hi)
    return "x".join(str(max(3, min(hi, int(round(s * rng.uniform(0.8, 1.2)))))) for _ in range(dim))


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "spmv", "multi", "smooth", "mg", "assemble", "parts", "serve"])
    if kind == "solve":
        box = rng.random() < 0.3
        dim = 3 if box else rng.choice([2, 3])
        grid = _grid(rng, dim, 8, 100) if box else _grid(rng, dim, 12, 400 if dim == 2 else 128)
        return {"kind": kind, "grid": grid, "stencil": "box" if box else "axis",
                "precision": rng.choice(["fp64", "fp64", "mixed"])}
    if kind == "spmv":
        return {"kind": kind, "n": int(math.exp(rng.uniform(math.log(3e4), math.log(4e6)))),
                "precision": rng.choice(["fp64", "fp64", "fp32"])}
    if kind == "multi":
        return {"kind": kind, "grid": _grid(rng, 3, 16, 110), "k": rng.choice([2, 4, 8, 16])}
    if kind == "smooth":
        dim = rng.choice([2, 3])
        return {"kind": kind, "grid": _grid(rng, dim, 16, 1500 if dim == 2 else 140), "steps": rng.randint(1, 8),
                "residual": rng.random() < 0.3}
    if kind == "mg":
        return {"kind": kind, "grid": _grid(rng, 3, 20, 128), "precision": rng.choice(["fp64", "mixed"]),
                "cycle": rng.choice([1, 1, 2])}
    if kind == "assemble":
        return {"kind": kind, "grid": _grid(rng, 3, 16, 110), "mg": rng.random() < 0.5}
    if kind == "parts":
        return {"kind": kind, "grid": _grid(rng, 3, 10, 160)}
    return {"kind": kind, "count": rng.randint(4, 20), "mix": rng.randrange(1, 1 << 20), "side2d": 256, "side3d": 64}


# ------------------------------------------------------------------ inputs
def _shape(case):
    return [int(v) for v in case["grid"].split("x")]  # first extent fastest


def _rand(n, seed, k=None):
    """Uniform in [-1, 1), n entries or an n x k block."""
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * seed + 17)
    return torch.rand(n if k is None else (n, k), generator=g, device=DEV, dtype=torch.float64) * 2 - 1


def _offsets(dim, stencil):
    """Neighbour steps (z, y, x) in ascending column order, the diagonal among them."""
    r = [(c, b, a) for c in ((-1, 0, 1) if dim > 2 else (0,)) for b in (-1, 0, 1) for a in (-1, 0, 1)]
    return r if stencil == "box" else [o for o in r if sum(map(abs, o)) <= 1]


def _coefficients(case, seed):
    """One (nz, ny, nx) array per neighbour step: the matrix entries, zero where
    the step leaves the grid.  axis: the unscaled Dirichlet Laplacian (2 dim on
    the diagonal, -1 beside it); box: 27-point diffusion, symmetric lognormal
    weights, those that leave the grid on the diagonal only."""
    s = _shape(case)
    dim = len(s)
    nx, ny, nz = s[0], s[1], s[2] if dim > 2 else 1
    steps = _offsets(dim, case.get("stencil", "axis"))
    full = (nz, ny, nx)

    def inside(o):
        return tuple(slice(max(0, -d), n - max(0, d)) for d, n in zip(o, full))

    out = {}
    if case.get("stencil", "axis") == "axis":
        for o in steps:
            a = torch.zeros(full, device=DEV, dtype=torch.float64)
            a[inside(o)] = 2.0 * dim if o == (0, 0, 0) else -1.0
            out[o] = a
        return steps, out
    g = torch.Generator(device=DEV)
    g.manual_seed(7919 * seed + 5)
    diag = torch.zeros(full, device=DEV, dtype=torch.float64)
    for o in steps:
        if o <= (0, 0, 0):
            continue
        back = tuple(-d for d in o)
        w = torch.randn(full, generator=g, device=DEV, dtype=torch.float64).exp()
        beyond = torch.randn(full, generator=g, device=DEV, dtype=torch.float64).exp()
        up, down = torch.zeros_like(w), torch.zeros_like(w)
        up[inside(o)] = -w[inside(o)]
        down[inside(back)] = -w[inside(o)]
        out[o], out[back] = up, down
        diag += w
        diag += torch.where(down == 0, beyond, -down)
    out[(0, 0, 0)] = diag
    return steps, out


def _csr(case, seed):
    """(rowptr, col, val) on the GPU, columns ascending in each row."""
    s = _shape(case)
    nx, ny = s[0], s[1]
    steps, coef = _coefficients(case, seed)
    n = math.prod(s)
    val = torch.stack([coef[o].reshape(-1) for o in steps], dim=1)
    del coef
    shift = torch.tensor([(o[0] * ny + o[1]) * nx + o[2] for o in steps], device=DEV, dtype=torch.int64)
    keep = val != 0
    col = (torch.arange(n, device=DEV, dtype=torch.int64)[:, None] + shift[None, :]).to(torch.int32)[keep]
    rowptr = torch.zeros(n + 1, device=DEV, dtype=torch.int64)
    rowptr[1:] = keep.sum(dim=1).cumsum(0)
    return rowptr.to(torch.int32), col, val[keep]


def _powerlaw(n, seed):
    """(rowptr, col, val): zipf(1.8) picks per row in [3, 4000], uniform columns,
    symmetrised, one normal value per pair, a dominant diagonal.  Values are
    multiples of 2^-20, so that the row sums are exact in any order."""
    g = torch.Generator(device=DEV)
    g.manual_seed(104729 * seed + 3)
    top = 4000
    pick = torch.arange(1, 1 << 16, device=DEV, dtype=torch.float64) ** -1.8
    u = torch.rand(n, generator=g, device=DEV, dtype=torch.float64)
    d = (torch.searchsorted((pick.cumsum(0) / pick.sum()).contiguous(), u) + 1).clamp(3, min(top, n - 1))
    i = torch.repeat_interleave(torch.arange(n, device=DEV), d)
    j = torch.randint(0, n, (i.numel(),), generator=g, device=DEV)
    key = torch.unique((torch.minimum(i, j) * n + torch.maximum(i, j))[i != j])
    del i, j, d, u
    a, b = key // n, key % n
    v = (torch.randn(key.numel(), generator=g, device=DEV, dtype=torch.float64) * 2 ** 20).round().to(torch.int64)
    v = torch.where(v == 0, torch.ones_like(v), v)
    total = torch.zeros(n, device=DEV, dtype=torch.int64)
    total.index_add_(0, a, v.abs()).index_add_(0, b, v.abs())
    r = torch.arange(n, device=DEV)
    keys, order = torch.sort(torch.cat([a * n + b, b * n + a, r * n + r]))
    val = torch.cat([v, v, total + 2 ** 20])[order].double() * 2.0 ** -20
    row = keys // n
    rowptr = torch.zeros(n + 1, device=DEV, dtype=torch.int64)
    rowptr[1:] = torch.bincount(row, minlength=n).cumsum(0)
    return rowptr.to(torch.int32), (keys % n).to(torch.int32), val


def _requests(case, seed):
    """The burst's systems: sides from the case, shifts and right-hand sides from the seed."""
    sides = spkgen.serve_stream(seed=case["mix"], count=case["count"], side2d=(32, case["side2d"]),
                                side3d=(16, case["side3d"]))
    rng = np.random.default_rng(seed)
    return [(spkgen.ServeRequest(0.0, q.dim, q.side, float(rng.uniform(0.0, 1.0)), 0),
             rng.uniform(-1.0, 1.0, q.n)) for q in sides]


# ------------------------------------------------------------------ a pass
def prepare(case, seed):
    kind = case["kind"]
    if kind == "serve":
        systems = []
        for q, b in _requests(case, seed):
            A = spkgen.serve_matrix(q)
            systems.append((A.rowptr, A.col, A.val, b))
        return {"kind": kind, "systems": systems, "server": spk.server_create(), "opts": spk.ksp_opts()}
    if kind == "spmv":
        f32 = case["precision"] == "fp32"
        M = spk.mat_create_csr(*_powerlaw(case["n"], seed), flags=spk.MAT_MIXED if f32 else 0)
        x = _rand(case["n"], seed)
        x = x.float() if f32 else x
        return {"kind": kind, "M": M, "x": x, "y": torch.zeros_like(x), "f32": f32}
    csr = _csr(case, seed)
    n = csr[0].numel() - 1
    state = {"kind": kind, "case": dict(case)}
    if kind == "assemble":
        b = _rand(n, seed)
        return state | {"csr": csr, "b": b, "x": torch.zeros_like(b), "shape": _shape(case), "mg": case["mg"]}
    mixed = case.get("precision") == "mixed"
    M = spk.mat_create_csr(*csr, flags=spk.MAT_MIXED if mixed else 0)
    b = _rand(n, seed, case.get("k"))
    state |= {"M": M, "b": b, "x": torch.zeros_like(b)}
    if kind == "solve":
        state["opts"] = spk.ksp_opts(precision=spk.PREC_MIXED if mixed else spk.PREC_FP64)
    elif kind == "smooth":
        state["r"] = torch.zeros_like(b) if case["residual"] else None
    elif kind == "mg":
        state["mg"] = spk.mg_create(M, _shape(case), spk.mg_opts(
            cycle=case["cycle"], precision=spk.PREC_MIXED if mixed else spk.PREC_FP64))
    elif kind == "parts":
        state |= {"q": torch.zeros_like(b), "z": torch.zeros_like(b), "p": _rand(n, seed + 500009),
                  "two": torch.zeros(2, device=DEV, dtype=torch.float64),
                  "norm": torch.zeros(1, device=DEV, dtype=torch.float64)}
    return state


def run(s):
    kind = s["kind"]
    if kind == "solve":
        spk.ksp_solve(s["M"], s["b"], s["x"], s["opts"])
        return {"x": s["x"]}
    if kind == "spmv":
        (spk.mat_mult_f32 if s["f32"] else spk.mat_mult)(s["M"], s["x"], s["y"])
        return {"y": s["y"]}
    if kind == "multi":
        spk.ksp_solve_multi(s["M"], s["b"], s["x"])
        return {"x": s["x"]}
    if kind == "smooth":
        spk.pc_chebyshev(s["M"], s["b"], s["x"], s["case"]["steps"], emin=0.2, emax=2.0, r_out=s["r"])
        return {"x": s["x"], "r": s["r"]}
    if kind == "mg":
        spk.ksp_solve_mg(s["mg"], s["b"], s["x"])
        return {"x": s["x"]}
    if kind == "assemble":
        with spk.mat_create_csr(*s["csr"]) as M:
            if s["mg"]:
                with spk.mg_create(M, s["shape"]) as H:
                    spk.ksp_solve_mg(H, s["b"], s["x"])
            else:
                spk.mat_mult(M, s["b"], s["x"])
        return {"x": s["x"]}
    if kind == "parts":
        M, p, q, z = s["M"], s["p"], s["q"], s["z"]
        spk.mat_mult(M, p, q)                # q = A p
        spk.vec_dot2(p, q, s["b"], s["two"])  # p.q and p.r
        spk.pc_jacobi_apply(M, s["b"], z)    # z = D^-1 r
        spk.vec_axpy(-0.375, q, z)           # z -= alpha q
        spk.vec_aypx(0.625, p, q)            # q = p + beta q
        spk.vec_nrm2(z, s["norm"])
        return {"z": z, "q": q, "dots": s["two"], "norm": s["norm"]}
    S, out = s["server"], {}
    where = {}
    for i, (rowptr, col, val, b) in enumerate(s["systems"]):
        where[spk.server_submit(S, rowptr, col, val, b, s["opts"])] = i
    while len(out) < len(where):
        spk.server_progress(S, 1)
        for t in spk.server_completed(S):
            x = np.empty(len(s["systems"][where[t]][3]))
            spk.server_poll(S, t, x)
            out[where[t]] = x
    return {"x": np.concatenate([out[i] for i in range(len(out))])}


# ------------------------------------------------------------------ what a pass cannot do without
def _entries(case):
    """(rows, stored entries) of a grid matrix."""
    s = _shape(case)
    n = math.prod(s)
    if case.get("stencil", "axis") == "box":
        return n, math.prod(3 * v - 2 for v in s)
    return n, n + 2 * sum(n // v * (v - 1) for v in s)


def work(case):
    """Matrix and right-hand sides read once and results written once for each
    pass; solves: that for each iteration of the usual count (no more than an
    estimate from the grid's extent), the matrix once and the five Krylov
    vectors of each."""
    kind = case["kind"]
    if kind == "serve":
        by = fl = 0.0
        for q, _ in _requests(case, 0):
            nnz = (2 * q.dim + 1) * q.n
            its = 2.0 * min(q.side, 60)
            by += 12.0 * nnz + 20.0 * q.n
            fl += its * (2.0 * nnz + 12.0 * q.n)
        return {"bytes": by, "flops": fl}
    if kind == "spmv":
        n, w = case["n"], 8 if case["precision"] == "fp64" else 4
        nnz = 33.3 * n
        return {"bytes": (w + 4) * nnz + 4 * n + 2 * w * n, "flops": 2 * nnz}
    n, nnz = _entries(case)
    csr = 12 * nnz + 4 * (n + 1)
    if kind == "solve":
        its = 3.0 * max(_shape(case)) if case["stencil"] == "axis" else 2.4 * max(_shape(case))
        w = 8 if case["precision"] == "fp64" else 4
        return {"bytes": its * ((w + 4) * nnz + 11 * w * n), "flops": its * (2 * nnz + 12 * n)}
    if kind == "multi":
        its, k = 3.0 * max(_shape(case)), case["k"]
        return {"bytes": its * (csr + 88 * n * k), "flops": its * k * (2 * nnz + 12 * n)}
    if kind == "smooth":
        passes = case["steps"] - (0 if case["residual"] else 1)
        return {"bytes": max(1, passes) * csr + 24 * n, "flops": passes * 2 * nnz + 6 * n * case["steps"]}
    if kind == "mg":
        return {"bytes": 14 * (5 * csr + 88 * n), "flops": 14 * (5 * 2 * nnz + 40 * n)}
    if kind == "assemble":
        if case["mg"]:
            return {"bytes": 14 * (5 * csr + 88 * n), "flops": 14 * (5 * 2 * nnz + 40 * n)}
        return {"bytes": csr + 16 * n, "flops": 2 * nnz}
    return {"bytes": csr + 48 * n, "flops": 2 * nnz + 13 * n}


# ------------------------------------------------------------------ 64-bit results
def _apply(steps, coef, x):
    """A x on the grid, in the columns' order."""
    y = torch.zeros_like(x)
    for o in steps:
        src = tuple(slice(max(0, d), n + min(0, d)) for d, n in zip(o, x.shape))
        dst = tuple(slice(max(0, -d), n - max(0, d)) for d, n in zip(o, x.shape))
        y[dst] += coef[o][dst] * x[src]
    return y


def _sine_solve(b, shape, shift=0.0):
    """(Laplacian + shift)^-1 b by sine transforms; b is (n,) or (n, k), first extent fastest."""
    k = b.shape[1] if b.dim() == 2 else 1
    t = b.reshape(*reversed(shape), k)
    lam = torch.full((1,) * len(shape) + (1,), float(shift), device=b.device, dtype=torch.float64)
    mats = []
    for axis, n in enumerate(reversed(shape)):
        m = torch.arange(1, n + 1, device=b.device, dtype=torch.float64)
        mats.append(torch.sin(m[:, None] * m[None, :] * (math.pi / (n + 1))) * math.sqrt(2.0 / (n + 1)))
        at = [1] * (len(shape) + 1)
        at[axis] = n
        lam = lam + (2 - 2 * torch.cos(m * (math.pi / (n + 1)))).reshape(at)

    def transform(t):
        for axis, S in enumerate(mats):
            t = torch.tensordot(S, t, dims=([1], [axis])).movedim(0, axis)
        return t

    return transform(transform(t) / lam).reshape(b.shape)


def _cg_solve(steps, coef, b):
    """Jacobi-PCG in 64 bits to the accuracy that 64 bits give."""
    dinv = 1.0 / coef[(0, 0, 0)]
    x, r = torch.zeros_like(b), b.clone()
    z = dinv * r
    p, rho, stop = z.clone(), (r * z).sum(), 1e-13 * b.norm()
    for k in range(5000):
        q = _apply(steps, coef, p)
        a = rho / (p * q).sum()
        x += a * p
        r -= a * q
        if k % 50 == 49 and r.norm() <= stop:
            break
        z = dinv * r
        new = (r * z).sum()
        p = z + (new / rho) * p
        rho = new
    return x


def _smooth(steps, coef, b, count, emin, emax):
    """x and b - A x after `count` Chebyshev-Jacobi steps from zero."""
    dinv = 1.0 / coef[(0, 0, 0)]
    theta, delta = 0.5 * (emax + emin), 0.5 * (emax - emin)
    sigma = theta / delta
    x, r = torch.zeros_like(b), b.clone()
    d, rho = dinv * r / theta, 1.0 / sigma
    for _ in range(count):
        x = x + d
        r = r - _apply(steps, coef, d)
        new = 1.0 / (2.0 * sigma - rho)
        d = new * rho * d + (2.0 * new / delta) * (dinv * r)
        rho = new
    return x, r


def exact(case, seed):
    kind = case["kind"]
    if kind == "serve":
        out = []
        for q, b in _requests(case, seed):
            out.append(_sine_solve(torch.from_numpy(b).to(DEV), [q.side] * q.dim, q.shift).cpu().numpy())
        return {"x": np.concatenate(out)}
    if kind == "spmv":
        rowptr, col, val = _powerlaw(case["n"], seed)
        x = _rand(case["n"], seed)
        if case["precision"] == "fp32":
            val, x = val.float().double(), x.float().double()
        row = torch.repeat_interleave(torch.arange(case["n"], device=DEV), rowptr.diff().long())
        return {"y": torch.zeros_like(x).index_add_(0, row, val * x[col.long()])}
    n = math.prod(_shape(case))
    b = _rand(n, seed, case.get("k"))
    if kind in ("mg", "multi") or (kind == "solve" and case["stencil"] == "axis") or (
            kind == "assemble" and case["mg"]):
        return {"x": _sine_solve(b, _shape(case))}
    steps, coef = _coefficients(case, seed)
    full = coef[(0, 0, 0)].shape
    if kind == "solve":
        return {"x": _cg_solve(steps, coef, b.reshape(full)).reshape(-1)}
    if kind == "assemble":
        return {"x": _apply(steps, coef, b.reshape(full)).reshape(-1)}
    if kind == "smooth":
        x, r = _smooth(steps, coef, b.reshape(full), case["steps"], 0.2, 2.0)
        return {"x": x.reshape(-1), "r": r.reshape(-1) if case["residual"] else None}
    p = _rand(n, seed + 500009)
    q = _apply(steps, coef, p.reshape(full)).reshape(-1)
    z = b / coef[(0, 0, 0)].reshape(-1) - 0.375 * q
    return {"z": z, "q": p + 0.625 * q, "dots": torch.stack([(p * q).sum(), (p * b).sum()]), "norm": z.norm()[None]}
