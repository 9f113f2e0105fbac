"""Timing cases of the library: what a program that solves sparse systems has it do.

Each case is one call (or the few calls that belong together) of the Python binding
``paper_1606_00545_amd.hec`` on inputs of a stated shape. Kinds:

* ``spmv``  -- y = A x with a resident matrix (HEC, plain CSR or HYB layout);
* ``trsv``  -- the preconditioner solve x = U^{-1} L^{-1} b of a resident ILU(k) factor;
* ``solve`` -- a whole Krylov solve (GMRES(30) or BiCGSTAB) on resident handles;
* ``batch`` -- many small systems solved by GMRES(30) in one call (the serving path);
* ``amg``   -- a whole AMG solve on a resident hierarchy;
* ``setup`` -- a new matrix on the host made ready to solve with: matrix, factor and
  schedules built, the factor's values read back.

Matrices are those of ``synth.py``: constant-coefficient Poisson and lognormal
two-point-flux stencils on 2D and 3D grids, and power-law random rows.
"""
import math

import numpy as np
import torch

from paper_1606_00545_amd import hec, synth


# ------------------------------------------------------------------ cases

def listed():
    return [
        # one product with a small 2D stencil matrix: nothing but call and launch latency
        dict(name="spmv_poisson64", kind="spmv", mat="grid", nx=64, ny=64, nz=1, sigma=0.0, zscale=1.0,
             fmt="hec", vals="f64"),
        # the product inside every Krylov iteration of a 2.1M-row reservoir-like system
        dict(name="spmv_tpfa128", kind="spmv", mat="grid", nx=128, ny=128, nz=128, sigma=2.0, zscale=1.0,
             fmt="hec", vals="f64"),
        # irregular rows (4..512 entries): ELL part and CSR remainder, random gathers
        dict(name="spmv_powerlaw300k", kind="spmv", mat="powerlaw", n=300_000, fmt="hec", vals="f64"),
        # ILU(0) preconditioner solve of the 2.1M-row 3D system
        dict(name="trsv_tpfa128", kind="trsv", mat="grid", nx=128, ny=128, nz=128, sigma=2.0, zscale=1.0, k=0,
             vals="f64"),
        # the same in 2D on a ragged grid: the longest level chains among the serving requests
        dict(name="trsv_2d_701x653", kind="trsv", mat="grid", nx=701, ny=653, nz=1, sigma=1.5, zscale=1.0, k=0,
             vals="f64"),
        # ILU(1) with FP32 values: the preconditioner of the mixed-precision inner solve (layered medium)
        dict(name="trsv_ilu1_f32", kind="trsv", mat="grid", nx=75, ny=62, nz=51, sigma=2.0, zscale=0.01, k=1,
             vals="f32"),
        # ILU(0) of an irregular matrix: rows too long for the slab of the blocked solve
        dict(name="trsv_powerlaw60k", kind="trsv", mat="powerlaw", n=60_000, k=0, vals="f64"),
        # a whole small solve: 4096 rows, bound by latency and launches
        dict(name="gmres_poisson64", kind="solve", method="gmres", nx=64, ny=64, nz=1, sigma=0.0, rtol=1e-8),
        # a whole large solve: the 128^3 system of the benchmark
        dict(name="gmres_tpfa128", kind="solve", method="gmres", nx=128, ny=128, nz=128, sigma=2.0, rtol=1e-8),
        # 48 small systems of 1000 to 4200 rows, half 2D, half 3D, as a server collects them
        dict(name="batch48", kind="batch", count=48, nmin=1000, nmax=4200, sigma=1.5, rtol=1e-8),
        # the paper's AMG configuration: 3D Poisson 50^3, damped Jacobi 3 + 3, to 1e-8
        dict(name="amg_poisson50", kind="amg", nx=50, ny=50, nz=50, sigma=0.0, smoother="jacobi", rtol=1e-8),
        # a request with a new matrix: everything before its first solve
        dict(name="setup_tpfa60", kind="setup", nx=60, ny=60, nz=60, sigma=2.0, k=0),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _grid_shape(rng, nmin, nmax, dim=None):
    """A 2D or 3D grid of about log-uniform size whose edges differ."""
    dim = dim or rng.choice((2, 3))
    n = math.exp(rng.uniform(math.log(nmin), math.log(nmax)))
    e = n ** (1.0 / dim)
    edges = [max(17, int(e * rng.uniform(0.8, 1.25))) if dim == 2 else max(9, int(e * rng.uniform(0.85, 1.15)))
             for _ in range(dim)]
    while math.prod(edges) > nmax:
        edges[0] = max(9, edges[0] - 1)
        edges[-1] = max(9, edges[-1] - 1)
    return dict(nx=edges[0], ny=edges[1], nz=edges[2] if dim == 3 else 1)


def draw(rng):
    kind = rng.choice(("spmv", "spmv", "trsv", "trsv", "trsv", "solve", "batch", "amg", "setup"))
    if kind == "spmv":
        fmt, vals = rng.choice(("hec", "hec", "csr", "hyb")), rng.choice(("f64", "f64", "f32"))
        if rng.random() < 0.4:
            return dict(kind=kind, mat="powerlaw", n=_logint(rng, 5_000, 300_000), fmt=fmt, vals=vals)
        return dict(kind=kind, mat="grid", **_grid_shape(rng, 4_000, 2_000_000), sigma=round(rng.uniform(0.5, 3), 2),
                    zscale=1.0, fmt=fmt, vals=vals)
    if kind == "trsv":
        vals = rng.choice(("f64", "f64", "f32"))
        if rng.random() < 0.25:
            return dict(kind=kind, mat="powerlaw", n=_logint(rng, 5_000, 60_000), k=0, vals=vals)
        k = rng.choice((0, 0, 0, 1, 2, 3))
        shape = _grid_shape(rng, 1_000, 1_500_000 if k == 0 else 250_000 if k == 1 else 60_000)
        return dict(kind=kind, mat="grid", **shape, sigma=round(rng.uniform(0.5, 3), 2),
                    zscale=rng.choice((1.0, 0.01)), k=k, vals=vals)
    if kind == "solve":
        if rng.random() < 0.25:  # a well-conditioned system asked for all its digits
            return dict(kind=kind, method="bicgstab", **_grid_shape(rng, 4_000, 200_000, 3),
                        sigma=round(rng.uniform(0.2, 0.8), 2), rtol=1e-12)
        return dict(kind=kind, method="gmres", **_grid_shape(rng, 1_000, 300_000, 3 if rng.random() < 0.6 else 2),
                    sigma=round(rng.uniform(0.5, 2), 2), rtol=1e-8)
    if kind == "batch":
        return dict(kind=kind, count=_logint(rng, 4, 64), nmin=1000, nmax=_logint(rng, 1500, 8000),
                    sigma=round(rng.uniform(0.5, 2), 2), rtol=1e-8)
    if kind == "amg":
        return dict(kind=kind, **_grid_shape(rng, 5_000, 150_000), sigma=rng.choice((0.0, round(rng.uniform(0.5, 2), 2))),
                    smoother=rng.choice(("jacobi", "jacobi", "chebyshev")), rtol=1e-8)
    return dict(kind=kind, **_grid_shape(rng, 1_000, 300_000), sigma=round(rng.uniform(0.5, 3), 2),
                k=rng.choice((0, 0, 1)))


# ------------------------------------------------------------------ inputs

def _matrix(case, rng):
    if case.get("mat") == "powerlaw":
        return synth.powerlaw_random(case["n"], rng)
    shape = (case["nx"], case["ny"]) if case["nz"] == 1 else (case["nx"], case["ny"], case["nz"])
    if case["sigma"] == 0.0:  # constant coefficients: the Poisson stencils of synth.py
        return synth.poisson2d(shape[0]) if len(set(shape)) == 1 and len(shape) == 2 else \
            synth.poisson3d(shape[0]) if len(set(shape)) == 1 else _lognormal(shape, 0.0, 1.0, rng)
    return _lognormal(shape, case["sigma"], case.get("zscale", 1.0), rng)


def _lognormal(shape, sigma, zscale, rng):
    return synth.lognormal_tpfa(shape, sigma, rng, zscale=zscale)


def _batch_matrices(case, rng):
    """2D and 3D systems in turn, their sizes spread evenly in the logarithm from nmin to nmax."""
    for i in range(case["count"]):
        n = case["nmin"] * (case["nmax"] / case["nmin"]) ** ((i + 0.5) / case["count"])
        dim = 2 + i % 2
        m = max(2, int(n ** (1.0 / dim)))
        A = synth.lognormal_tpfa((m,) * dim, case["sigma"], rng)
        yield A, synth.uniform_vector(A.n, rng)


def _system(A, xt, k=0, keep_f32=False):
    """Matrix, factor, schedules and b = A x_true, all resident."""
    M = hec.hec_from_csr(A, keep_f32=keep_f32)
    F = hec.ilu_factor(A, k=k, keep_f32=keep_f32)
    lv = hec.level_schedule(F)
    b = torch.empty(A.n, dtype=torch.float64, device="cuda")
    hec.hec_spmv(M, torch.from_numpy(xt).cuda(), b)
    return M, F, lv, b, torch.empty_like(b)


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    kind = case["kind"]
    if kind == "batch":
        systems = [_system(A, xt) for A, xt in _batch_matrices(case, rng)]
        B = hec.Batch(case["count"], restart=30, max_n=max(s[0].n for s in systems))
        torch.cuda.synchronize()
        return kind, case, (B, systems)
    A = _matrix(case, rng)
    if kind == "setup":
        return kind, case, (A,)
    xt = synth.uniform_vector(A.n, rng)
    if kind == "spmv":
        f32 = case["vals"] == "f32"
        if case["fmt"] == "hyb":
            M = hec.hec_from_csr(A, ell_width=hec.WIDTH_HYB, coo=True, keep_f32=f32)
        else:
            M = hec.hec_from_csr(A, ell_width=0 if case["fmt"] == "csr" else -1, keep_f32=f32)
        x = torch.from_numpy(xt).cuda().to(torch.float32 if f32 else torch.float64)
        return kind, case, (M, x, torch.empty_like(x), hec.F32 if f32 else hec.F64)
    if kind == "trsv":
        f32 = case["vals"] == "f32"
        F = hec.ilu_factor(A, k=case["k"], keep_f32=f32)
        lv = hec.level_schedule(F)
        b = torch.from_numpy(xt).cuda().to(torch.float32 if f32 else torch.float64)
        return kind, case, (F, lv, b, torch.empty_like(b))
    if kind == "solve":
        return kind, case, _system(A, xt)
    H = hec.amg_setup(A, smoother=case["smoother"])
    M = hec.hec_from_csr(A)
    b = torch.empty(A.n, dtype=torch.float64, device="cuda")
    hec.hec_spmv(M, torch.from_numpy(xt).cuda(), b)
    return kind, case, (H, b, torch.empty_like(b))


# ------------------------------------------------------------------ one pass

def run(state):
    kind, case, s = state
    if kind == "spmv":
        M, x, y, vals = s
        return hec.hec_spmv(M, x, y, vals=vals)
    if kind == "trsv":
        F, lv, b, x = s
        return hec.trsv_levels(F, lv, b, x)
    if kind == "solve":
        M, F, lv, b, x = s
        if case["method"] == "gmres":
            hec.gmres_solve(M, F, lv, b, x, restart=30, rtol=case["rtol"])
        else:
            hec.bicgstab_solve(M, F, lv, b, x, rtol=case["rtol"])
        return x
    if kind == "batch":
        B, systems = s
        hec.gmres_solve_batched(B, systems, rtol=case["rtol"])
        return [sys[4] for sys in systems]
    if kind == "amg":
        H, b, x = s
        hec.amg_solve(H, b, x, rtol=case["rtol"])
        return x
    A, = s
    M = hec.hec_from_csr(A)
    F = hec.ilu_factor(A, k=case["k"])
    lv = hec.level_schedule(F)
    LUx = hec.ilu_export(F)[2]
    for h in (lv, F, M):
        h.close()
    return LUx


# ------------------------------------------------------------------ what a pass cannot do without

def _rows_nnz(case):
    if case.get("mat") == "powerlaw":
        return case["n"], 12 * case["n"]
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    n = nx * ny * nz
    return n, n + 2 * ((nx - 1) * ny * nz + nx * (ny - 1) * nz + nx * ny * (nz - 1))


def work(case):
    kind = case["kind"]
    if kind == "batch":
        # about 0.8 sqrt(n) (2D) and 0.9 n^(1/3) + 10 (3D) GMRES steps a system; the system stays in cache,
        # so its matrix, factor and vectors are read once: the operations are what is left
        total = flops = 0.0
        for i in range(case["count"]):
            n = math.sqrt(case["nmin"] * case["nmax"])
            nnz, its = (5 * n, 0.8 * math.sqrt(n)) if i % 2 == 0 else (7 * n, 0.9 * n ** (1 / 3) + 10)
            total += 24 * nnz + 16 * n
            flops += its * (4 * nnz + 8 * 15 * n)
        return {"bytes": total, "flops": flops}
    n, nnz = _rows_nnz(case)
    vb = 4 if case.get("vals") == "f32" else 8
    if kind == "spmv":
        return {"bytes": (vb + 4) * nnz + 2 * vb * n, "flops": 2 * nnz}
    if kind in ("trsv", "setup"):
        per = {2: (5, 7, 9, 13), 3: (7, 12.9, 22.7, 42.2)}[2 if case.get("nz", 2) == 1 else 3][case["k"]]
        lu = nnz if case["k"] == 0 else per * n
        if kind == "trsv":
            return {"bytes": (vb + 4) * lu + 4 * vb * n, "flops": 2 * lu}
        # the matrix in, its device form, the factor and the two solve plans out, the factor read back
        return {"bytes": 12 * nnz + 12 * nnz + 3 * 12 * lu + 8 * lu, "flops": 2 * lu * per / 2}
    if kind == "solve":
        e = n ** (1 / 3 if case["nz"] > 1 else 1 / 2)
        its = 1.17 * e if case["nz"] > 1 else 0.9 * e
        if case["method"] == "bicgstab":  # two products and two preconditioner solves a pass
            its *= 1.2
            return {"bytes": its * (24 * nnz + 200 * n), "flops": its * 8 * nnz}
        # per step: the product, the factor, two passes over half a full basis
        return {"bytes": its * (24 * nnz + 48 * n + 2 * 15 * 8 * n), "flops": its * (4 * nnz + 8 * 15 * n)}
    cycles, complexity = 6 if case["sigma"] == 0.0 else 15, 2.8 if case["nz"] > 1 else 2.2
    return {"bytes": cycles * 8 * complexity * (12 * nnz + 32 * n), "flops": cycles * 8 * complexity * 2 * nnz}


# ------------------------------------------------------------------ values in 64 bits, without the library

def _levels_grid(nx, ny, nz):
    """Cells grouped by x + y + z (the levels of an ILU(0) factor of the stencil)."""
    c = np.arange(nx * ny * nz)
    lev = c % nx + (c // nx) % ny + c // (nx * ny)
    order = np.argsort(lev, kind="stable")
    return np.split(order, np.cumsum(np.bincount(lev))[:-1])


def _stencil(A, nx, ny, nz):
    """The stencil's bands: {offset: a value per row, 0 where the neighbour does not exist}."""
    rows = np.repeat(np.arange(A.n), np.diff(A.Ap))
    out = {}
    for d in {0, 1, -1, nx, -nx} | ({nx * ny, -nx * ny} if nz > 1 else set()):
        m = A.Aj - rows == d
        out[d] = np.zeros(A.n)
        out[d][rows[m]] = A.Ax[m]
    return out


def _ilu0_stencil(A, nx, ny, nz):
    """ILU(0) of a 5- or 7-point stencil: bands of L (unit diagonal implied) and U, level by level.
    No entry besides the diagonal meets the product of two off-diagonal ones."""
    a = _stencil(A, nx, ny, nz)
    low = sorted(d for d in a if d < 0)
    L, diag = {d: a[d].copy() for d in low}, a[0].copy()
    for rows in _levels_grid(nx, ny, nz):
        for d in low:
            m = rows[L[d][rows] != 0]
            l = a[d][m] / diag[m + d]
            L[d][m] = l
            diag[m] -= l * a[-d][m + d]
    return L, diag, {-d: a[-d] for d in low}


def _solve_stencil(L, diag, U, b, nx, ny, nz):
    levels = _levels_grid(nx, ny, nz)
    x = b.astype(np.float64).copy()
    for rows in levels:
        for d in L:
            m = rows[L[d][rows] != 0]
            x[m] -= L[d][m] * x[m + d]
    for rows in reversed(levels):
        for d in U:
            m = rows[U[d][rows] != 0]
            x[m] -= U[d][m] * x[m + d]
        x[rows] /= diag[rows]
    return x


def _iluk_rows(A, k):
    """ILU(k), row by row: per row (columns, values) of L without its diagonal and of U with it."""
    Ap, Aj, Ax = A.Ap.tolist(), A.Aj.tolist(), A.Ax.tolist()
    upper, lower = [], []
    for i in range(A.n):
        val = dict(zip(Aj[Ap[i]:Ap[i + 1]], Ax[Ap[i]:Ap[i + 1]]))
        lev = dict.fromkeys(val, 0)
        todo = sorted(j for j in val if j < i)
        at = 0
        while at < len(todo):
            p = todo[at]
            at += 1
            pj, pv, pl = upper[p]
            l = val[p] / pv[0]
            val[p] = l
            lp = lev[p] + 1
            for j, v, jl in zip(pj[1:], pv[1:], pl[1:]):
                if j in val:
                    val[j] -= l * v
                    if lp + jl < lev[j]:
                        lev[j] = lp + jl
                elif lp + jl <= k:
                    val[j] = -l * v
                    lev[j] = lp + jl
                    if j < i:
                        todo.append(j)
                        todo[at:] = sorted(todo[at:])
        cols = sorted(val)
        cut = cols.index(i)
        lower.append((cols[:cut], [val[j] for j in cols[:cut]]))
        upper.append((cols[cut:], [val[j] for j in cols[cut:]], [lev[j] for j in cols[cut:]]))
    return lower, upper


def _solve_rows(lower, upper, b, f32):
    r = (lambda v: np.asarray(v, np.float32).tolist()) if f32 else (lambda v: v)
    x = b.tolist()
    for i, (cols, vals) in enumerate(lower):
        x[i] -= math.fsum(v * x[j] for j, v in zip(cols, r(vals)))
    for i in range(len(x) - 1, -1, -1):
        cols, vals, _ = upper[i]
        vals = r(vals)
        x[i] = (x[i] - math.fsum(v * x[j] for j, v in zip(cols[1:], vals[1:]))) / vals[0]
    return np.array(x)


def exact(case, seed):
    rng = np.random.default_rng(seed)
    kind = case["kind"]
    if kind == "batch":  # the solutions the right-hand sides were made from
        return [torch.from_numpy(xt) for _, xt in _batch_matrices(case, rng)]
    A = _matrix(case, rng)
    f32 = case.get("vals") == "f32"
    to32 = (lambda v: v.astype(np.float32).astype(np.float64)) if f32 else (lambda v: v)
    grid0 = case.get("mat") != "powerlaw" and case.get("k", 0) == 0
    if kind == "setup":
        if not grid0:
            if A.n * (1 + case["k"]) > 120_000:
                return None
            lower, upper = _iluk_rows(A, case["k"])
            return torch.tensor([v for lo, up in zip(lower, upper) for v in lo[1] + up[1]], dtype=torch.float64)
        L, diag, U = _ilu0_stencil(A, case["nx"], case["ny"], case["nz"])
        rows = np.repeat(np.arange(A.n), np.diff(A.Ap))
        out = np.empty(A.Ax.size)
        for d, v in {**L, 0: diag, **U}.items():
            m = A.Aj - rows == d
            out[m] = v[rows[m]]
        return torch.from_numpy(out)
    xt = synth.uniform_vector(A.n, rng)
    if kind == "spmv":
        return torch.from_numpy(np.add.reduceat(to32(A.Ax) * to32(xt)[A.Aj], A.Ap[:-1]))
    if kind == "trsv":
        if grid0:
            L, diag, U = _ilu0_stencil(A, case["nx"], case["ny"], case["nz"])
            L, U = {d: to32(v) for d, v in L.items()}, {d: to32(v) for d, v in U.items()}
            return torch.from_numpy(_solve_stencil(L, to32(diag), U, to32(xt), case["nx"], case["ny"], case["nz"]))
        if A.n * (1, 1, 3, 8)[case["k"]] > 250_000:
            return None  # row by row in plain Python: too long
        lower, upper = _iluk_rows(A, case["k"])
        return torch.from_numpy(_solve_rows(lower, upper, to32(xt), f32))
    return torch.from_numpy(xt)  # solves: the solution the right-hand side was made from
