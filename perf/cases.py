"""Timed cases of the library's main path: triangular solves and the preconditioners,
smoothers and Krylov solvers made of them, called through the Python binding.

A case is a dict of plain values.  ``kind`` names the entry point:

  tri       one lower triangular solve (tri_solve_lower) of an irregular matrix
  ilu       one ILU preconditioner application (ilu_apply), L then U
  ras       one block ILU (overlap 0) or RAS application (ras_apply)
  batch     one application of a batch of independent systems (batch_setup, ilu_apply)
  refactor  new values of A factored on the device, then one application
  sor       one symmetric SOR sweep (sor_apply)
  gmres     a whole GMRES(m) + ILU solve (krylov_solve)
  bicgstab  a whole BiCGSTAB + RAS solve with several right-hand sides

Grids are nx x ny x nz in natural order (nz = 1: two-dimensional five-point, else
seven-point).  sigma > 0: lognormal cell coefficients exp(sigma N(0,1)) from the seed,
harmonic means on the faces; sigma = 0: the Laplacian.  ``dtype`` is the type of the
factors, vectors are float64 (float32 for ``tri`` with float32 factors).  Right-hand
sides are U[-1, 1] from the seed.
"""
from __future__ import annotations

import functools
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_1606_00541_amd as H


def listed():
    return [
        # the smallest call: a 2D problem of a few thousand unknowns inside a time loop or as a
        # multigrid level; latency and launches count
        dict(name="ilu0_64x64", kind="ilu", nx=64, ny=64, nz=1, sigma=0.0, ilu="ilu0", k=0, dtype="f64", nrhs=1),
        # a general (not grid) lower triangle of odd size, single-precision solve with two
        # right-hand sides, as a user with their own factors calls it
        dict(name="tri_20011_f32_r2", kind="tri", n=20011, row=6, dtype="f32", nrhs=2),
        # an ordinary mid-size 3D problem on a ragged grid: ILU(1), FP32 factors for
        # refinement, four right-hand sides
        dict(name="ilu1_47x41x37_f32_r4", kind="ilu", nx=47, ny=41, nz=37, sigma=1.0, ilu="iluk", k=1, dtype="f32",
             nrhs=4),
        # a million unknowns with high contrast: ILUT(1e-3, 10), FP32 factors, long rows, thousands of levels
        dict(name="ilut_100cube_f32", kind="ilu", nx=100, ny=100, nz=100, sigma=2.0, ilu="ilut", p=10, tol=1e-3,
             dtype="f32", nrhs=1),
        # the benchmark's default system: ILU(0) of the 128^3 Laplacian in FP64
        dict(name="ilu0_128cube", kind="ilu", nx=128, ny=128, nz=128, sigma=0.0, ilu="ilu0", k=0, dtype="f64", nrhs=1),
        # block ILU(0) on 512 blocks of the 100^3 Laplacian (the paper's first example)
        dict(name="bilu0_100cube_512", kind="ras", nx=100, ny=100, nz=100, sigma=0.0, nsub=512, cut="box", overlap=0,
             dtype="f64", nrhs=1),
        # restricted additive Schwarz on 64 uneven contiguous subdomains, overlap 1, FP32
        # factors, 16 right-hand sides
        dict(name="ras_128cube_64_r16_f32", kind="ras", nx=128, ny=128, nz=128, sigma=0.0, nsub=64, cut="slab",
             overlap=1, dtype="f32", nrhs=16),
        # many independent systems of uneven size at once, ILU(1), FP32 factors, 8 right-hand sides (the largest)
        dict(name="batch256_ilu1_r8_f32", kind="batch", nsys=256, nmin=1000, nmax=100000, shapes=5, sigma=1.0,
             ilu="iluk", k=1, dtype="f32", nrhs=8),
        # a new matrix of the same pattern every time step: refactor on the device, then apply
        dict(name="refactor_100cube", kind="refactor", nx=100, ny=100, nz=100, sigma=1.0, ilu="ilu0", k=0,
             dtype="f64", nrhs=1),
        # one symmetric Gauss-Seidel sweep, a multigrid smoother's call
        dict(name="ssor_100cube", kind="sor", nx=100, ny=100, nz=100, sigma=0.0, omega=1.0, dtype="f64", nrhs=1),
        # a whole linear solve to 1e-10, one right-hand side
        dict(name="gmres30_ilu0_100cube", kind="gmres", nx=100, ny=100, nz=100, sigma=0.0, m=30, its=231,
             dtype="f64", nrhs=1),
        # a whole linear solve to 1e-10 with 16 right-hand sides, RAS in FP32
        dict(name="bicgstab_ras_64cube_r16", kind="bicgstab", nx=64, ny=64, nz=64, sigma=0.0, nsub=16, cut="slab",
             overlap=1, its=76, dtype="f32", nrhs=16),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _grid(rng, lo, hi, dims=(2, 3, 3)):
    """Uneven grid sides with a product of about lo..hi (log-uniform)."""
    n = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    d = rng.choice(dims)
    a, b = rng.uniform(0.7, 1.4), rng.uniform(0.7, 1.4)
    if d == 2:
        s = n ** 0.5
        return dict(nx=max(8, int(round(s * a))), ny=max(8, int(round(s / a))), nz=1)
    s = n ** (1.0 / 3.0)
    return dict(nx=max(5, int(round(s * a))), ny=max(5, int(round(s * b))), nz=max(5, int(round(s / a / b))))


def draw(rng):
    kind = rng.choice(["tri", "ilu", "ilu", "ilu", "ilu", "ras", "ras", "batch", "refactor", "sor", "gmres",
                       "bicgstab"])
    if kind == "tri":
        return dict(kind=kind, n=_log_int(rng, 300, 100000), row=rng.randint(1, 12), dtype=rng.choice(["f64", "f32"]),
                    nrhs=rng.choice([1, 1, 2, 3, 4]))
    if kind == "ilu":
        c = dict(kind=kind, **_grid(rng, 500, 1500000), sigma=rng.choice([0.0, 1.0, 2.0]))
        n = c["nx"] * c["ny"] * c["nz"]
        ilu = rng.choice(["ilu0", "ilu0", "iluk", "ilut"])
        c.update(ilu=ilu, **(dict(k=0) if ilu == "ilu0" else dict(k=1) if ilu == "iluk" else dict(p=rng.randint(5, 10),
                                                                                                  tol=1e-3)))
        c.update(dtype=rng.choice(["f64", "f32"]), nrhs=rng.choice([1, 1, 1, 2, 3, 4, 8]) if n < 400000 else 1)
        return c
    if kind == "ras":
        c = dict(kind=kind, **_grid(rng, 20000, 1000000, (3,)), sigma=rng.choice([0.0, 1.0]))
        return dict(c, nsub=_log_int(rng, 8, 512), cut="box", overlap=rng.choice([0, 1]),
                    dtype=rng.choice(["f64", "f32"]), nrhs=rng.choice([1, 1, 4, 8, 16]))
    if kind == "batch":
        return dict(kind=kind, nsys=_log_int(rng, 16, 256), nmin=1000, nmax=_log_int(rng, 4000, 40000),
                    shapes=rng.randint(1, 1 << 20), sigma=1.0, ilu=rng.choice(["ilu0", "iluk"]), k=1,
                    dtype=rng.choice(["f64", "f32"]), nrhs=rng.choice([1, 2, 4, 8]))
    if kind == "refactor":
        return dict(kind=kind, **_grid(rng, 5000, 1000000), sigma=1.0, ilu=rng.choice(["ilu0", "ilu0", "iluk"]), k=1,
                    dtype=rng.choice(["f64", "f32"]), nrhs=1)
    if kind == "sor":
        return dict(kind=kind, **_grid(rng, 2000, 1000000), sigma=rng.choice([0.0, 1.0]),
                    omega=rng.choice([1.0, 1.3, 1.5]), dtype="f64", nrhs=rng.choice([1, 1, 2]))
    c = dict(kind=kind, **_grid(rng, 8000, 200000, (3,)), sigma=0.0)
    its = int(0.8 * max(c["nx"], c["ny"], c["nz"])) + 10
    if kind == "gmres":
        return dict(c, m=rng.choice([20, 30]), its=2 * its, dtype=rng.choice(["f64", "f32"]), nrhs=rng.choice([1, 1, 2]))
    return dict(c, nsub=rng.choice([4, 8, 16]), cut="slab", overlap=1, its=its, dtype="f32", nrhs=rng.choice([4, 8, 16]))


# ---- inputs ----------------------------------------------------------------

def _csr(n, col, val, mask):
    """CSR of row-wise candidate entries (columns ascending) where mask holds."""
    rowptr = np.zeros(n + 1, np.int64)
    np.cumsum(mask.sum(axis=1), out=rowptr[1:])
    return SimpleNamespace(n=n, rowptr=rowptr.astype(np.int32), col=col[mask].astype(np.int32), val=val[mask])


def _stencil(nx, ny, nz, sigma, seed):
    """Five- or seven-point diffusion matrix with Dirichlet walls, natural order."""
    n = nx * ny * nz
    dims = [nx, ny] + ([nz] if nz > 1 else [])
    stride = [1, nx, nx * ny][: len(dims)]
    idx = np.arange(n, dtype=np.int64)
    pos = [(idx // s) % d for s, d in zip(stride, dims)]
    kap = np.exp(sigma * np.random.default_rng(seed).standard_normal(n)) if sigma > 0 else None
    w, mid = 2 * len(dims) + 1, len(dims)
    col = np.empty((n, w), np.int64)
    val = np.empty((n, w))
    mask = np.ones((n, w), bool)
    diag = np.zeros(n)
    for a, (s, d) in enumerate(zip(stride, dims)):
        for side, e, ok in ((-1, mid - 1 - a, pos[a] > 0), (1, mid + 1 + a, pos[a] < d - 1)):
            j = np.where(ok, idx + side * s, idx)
            col[:, e] = j
            mask[:, e] = ok
            if kap is None:
                val[:, e] = -1.0
                diag += 1.0
            else:
                face = 2.0 * kap * kap[j] / (kap + kap[j])  # at a wall j is the cell itself: its own coefficient
                val[:, e] = -face
                diag += face
    col[:, mid] = idx
    val[:, mid] = diag
    return _csr(n, col, val, mask)


@functools.lru_cache(maxsize=8)
def _laplacian(nx, ny, nz):
    return _stencil(nx, ny, nz, 0.0, 0)


def _matrix(c, seed):
    return _stencil(c["nx"], c["ny"], c["nz"], c["sigma"], seed) if c["sigma"] > 0 else _laplacian(c["nx"], c["ny"],
                                                                                                   c["nz"])


def _triangle(c, seed):
    """Irregular lower triangle: up to ``row`` off-diagonals a row, most of them near
    the diagonal and one in ten anywhere before it; diagonal U[1, 2]."""
    n, w = c["n"], c["row"]
    rng = np.random.default_rng(seed)
    i = np.arange(n)[:, None]
    near = i - 1 - np.floor(rng.exponential(96.0, (n, w))).astype(np.int64)
    far = np.floor(rng.uniform(0.0, 1.0, (n, w)) * i).astype(np.int64)
    j = np.sort(np.where(rng.uniform(0.0, 1.0, (n, w)) < 0.1, far, near), axis=1)
    ok = (j >= 0) & (j < i)
    ok[:, 1:] &= j[:, 1:] != j[:, :-1]
    v = rng.uniform(-1.0, 1.0, (n, w)) / w
    return _csr(n, np.concatenate([j, i], axis=1), np.concatenate([v, rng.uniform(1.0, 2.0, (n, 1))], axis=1),
                np.concatenate([ok, np.ones((n, 1), bool)], axis=1))


def _sizes(c):
    """Sides of the batch's systems: log-uniform sizes, 2D or 3D by a coin."""
    rng = np.random.default_rng(c["shapes"])
    out = []
    for _ in range(c["nsys"]):
        t = math.exp(rng.uniform(math.log(c["nmin"]), math.log(c["nmax"])))
        if rng.uniform() < 0.5:
            s = int(round(t ** 0.5))
            out.append((s, s, 1))
        else:
            s = int(round(t ** (1.0 / 3.0)))
            out.append((s, s, s))
    return out


def _batch(c, seed):
    mats = [_stencil(*s, c["sigma"], [seed, i]) for i, s in enumerate(_sizes(c))]
    base = np.cumsum([0] + [m.n for m in mats])
    nz = np.cumsum([0] + [int(m.rowptr[-1]) for m in mats])
    rp = np.concatenate([m.rowptr[:-1].astype(np.int64) + nz[i] for i, m in enumerate(mats)] + [nz[-1:]])
    col = np.concatenate([m.col + np.int32(base[i]) for i, m in enumerate(mats)])
    a = SimpleNamespace(n=int(base[-1]), rowptr=rp.astype(np.int32), col=col, val=np.concatenate([m.val for m in mats]))
    return a, base.astype(np.int32)


def _owner(c):
    """Subdomain of every cell: axis-aligned boxes by recursive bisection, or uneven
    contiguous ranges of the natural order."""
    nx, ny, nz, parts = c["nx"], c["ny"], c["nz"], c["nsub"]
    n = nx * ny * nz
    if c["cut"] == "slab":
        rng = np.random.default_rng(parts)
        lo = n // (4 * parts)
        size = lo + np.floor(rng.dirichlet(np.full(parts, 2.0)) * (n - parts * lo)).astype(np.int64)
        size[-1] += n - size.sum()
        return np.repeat(np.arange(parts, dtype=np.int32), size)
    owner = np.empty((nz, ny, nx), np.int32)

    def rec(box, first, k):
        if k == 1:
            owner[tuple(slice(a, b) for a, b in box)] = first
            return
        ax = int(np.argmax([b - a for a, b in box]))
        lo, hi = box[ax]
        cut = lo + min(max(1, int(round((hi - lo) * (k // 2) / k))), hi - lo - 1)
        for part, f, m in (((lo, cut), first, k // 2), ((cut, hi), first + k // 2, k - k // 2)):
            sub = list(box)
            sub[ax] = part
            rec(sub, f, m)

    rec([(0, nz), (0, ny), (0, nx)], 0, parts)
    return owner.ravel()


def _rhs(n, nrhs, seed, dtype=torch.float64):
    b = np.random.default_rng([seed, 1]).uniform(-1.0, 1.0, (n, nrhs))
    return b, torch.from_numpy(b).to(dtype).cuda()


def _fill(c):
    return dict(k=c.get("k", 0), tol=c.get("tol", 0.0), p=c.get("p", 0))


def prepare(case, seed):
    c = case
    s = SimpleNamespace(kind=c["kind"], nrhs=c["nrhs"])
    tune = H.tune_default(max_nrhs=c["nrhs"])
    if c["kind"] == "tri":
        t = _triangle(c, seed)
        s.plan = H.tri_analyze(t, "lower", dtype=c["dtype"], tune=tune)
        s.b = _rhs(t.n, c["nrhs"], seed, torch.float32 if c["dtype"] == "f32" else torch.float64)[1]
        s.x = torch.empty_like(s.b)
        return s
    if c["kind"] == "batch":
        a, sys_ptr = _batch(c, seed)
        s.f = H.batch_setup(a, sys_ptr, c["ilu"], factor_dtype=c["dtype"], tune=tune, **_fill(c))
    else:
        a = _matrix(c, seed)
        if c["kind"] in ("ras", "bicgstab"):
            s.f = H.ras_setup(a, c["nsub"], _owner(c), overlap=c["overlap"], factor_dtype=c["dtype"], tune=tune)
        elif c["kind"] == "sor":
            s.f = H.sor_setup(a, c["omega"], tune=tune)
        elif c["kind"] == "refactor":
            # set up once on the Laplacian; the pattern's device maps belong to the handle
            first = _laplacian(c["nx"], c["ny"], c["nz"])
            s.f = H.ilu_setup(first, c["ilu"], factor_dtype=c["dtype"], tune=tune, **_fill(c))
            H.ilu_refactor(s.f, first)
            s.val = torch.from_numpy(a.val).cuda()
        else:
            s.f = H.ilu_setup(a, c.get("ilu", "ilu0"), factor_dtype=c["dtype"], tune=tune, **_fill(c))
    s.b = _rhs(a.n, c["nrhs"], seed)[1]
    s.x = torch.zeros_like(s.b)
    if c["kind"] in ("gmres", "bicgstab"):
        s.a = H.hec_from_csr(a)
        s.m = c.get("m", 30)
        s.method = "bicgstab" if c["kind"] == "bicgstab" else "gmres" if c["dtype"] == "f64" else "fgmres"
    return s


def run(state):
    s = state
    if s.kind == "tri":
        H.tri_solve_lower(s.plan, s.b, s.x)
    elif s.kind in ("ilu", "batch"):
        H.ilu_apply(s.f, s.b, s.x)
    elif s.kind == "ras":
        H.ras_apply(s.f, s.b, s.x)
    elif s.kind == "refactor":
        H.ilu_refactor(s.f, val=s.val)
        H.ilu_apply(s.f, s.b, s.x)
    elif s.kind == "sor":
        s.x.zero_()  # the smoother's initial guess
        H.sor_apply(s.f, s.b, s.x, sweeps=1, symmetric=True)
    else:
        s.x.zero_()
        H.krylov_solve(s.a, s.f, s.b, s.x, method=s.method, m=s.m, rtol=1e-10)
    return s.x


# ---- what a pass cannot do without -----------------------------------------

def _neighbours(c):
    """Unknowns and off-diagonal entries of one triangle of the grid's matrix."""
    if c["kind"] == "batch":
        shapes = _sizes(c)
    else:
        shapes = [(c["nx"], c["ny"], c["nz"])]
    n = off = 0
    for nx, ny, nz in shapes:
        m = nx * ny * nz
        n += m
        off += (nx - 1) * ny * nz + nx * (ny - 1) * nz + (nx * ny * (nz - 1) if nz > 1 else 0)
    return n, off


def work(case):
    c = case
    R, sv = c["nrhs"], 8 if c["dtype"] == "f64" else 4
    if c["kind"] == "tri":
        off = c["n"] * c["row"]
        return {"bytes": off * (sv + 4) + c["n"] * sv + 2 * c["n"] * R * sv, "flops": (2 * off + c["n"]) * R}
    n, off = _neighbours(c)
    fac = off  # off-diagonals of one factor
    if c.get("ilu") == "iluk":
        fac = 2 * off if c.get("nz", 2) > 1 else int(1.5 * off)  # the level-1 fill diagonals
    elif c.get("ilu") == "ilut":
        fac = n * c["p"]
    vec = 8 * n * R
    apply_b = 2 * fac * (sv + 4) + n * sv + 2 * vec
    apply_f = (4 * fac + n) * R
    if c["kind"] in ("ilu", "batch", "ras"):
        return {"bytes": apply_b, "flops": apply_f}
    if c["kind"] == "refactor":  # A's values in, factors out, then one application
        return {"bytes": 8 * (2 * off + n) + sv * (2 * fac + n) + apply_b, "flops": apply_f + 6 * n * 3}
    if c["kind"] == "sor":  # the matrix once per half sweep, b twice, x in and out
        return {"bytes": 2 * (2 * off + n) * 12 + 4 * vec, "flops": 2 * (4 * off + 2 * n) * R}
    mat = (2 * off + n) * 12
    if c["kind"] == "gmres":  # per iteration: M, A, and the basis read once for orthogonalization
        it_b, it_f = apply_b + mat + 2 * vec + (c["m"] // 2) * vec, apply_f + (4 * off + 2 * n + 2 * c["m"] * n) * R
    else:  # two applications, two products, the vectors of the recurrence
        it_b, it_f = 2 * apply_b + 2 * (mat + 2 * vec) + 10 * vec, 2 * apply_f + (8 * off + 24 * n) * R
    return {"bytes": c["its"] * it_b, "flops": c["its"] * it_f}


# ---- 64-bit values in plain numpy --------------------------------------------

def _ell(a):
    """Row-padded columns (padding n) and values [n][w] of a CSR matrix."""
    n, ln = a.n, np.diff(a.rowptr)
    w = int(ln.max())
    col = np.full((n, w), n, np.int64)
    val = np.zeros((n, w))
    at = np.arange(w)[None, :] < ln[:, None]
    col[at] = a.col
    val[at] = a.val
    return col, val


def _levels(col):
    """Rows grouped by dependency level; col [n][w] the off-diagonals, padding n."""
    n = col.shape[0]
    rows, slot = np.nonzero(col < n)
    dep = col[rows, slot]
    order = np.argsort(dep, kind="stable")
    child = rows[order]
    ptr = np.zeros(n + 1, np.int64)
    np.cumsum(np.bincount(dep, minlength=n), out=ptr[1:])
    left = np.bincount(rows, minlength=n)
    front, out = np.nonzero(left == 0)[0], []
    while front.size:
        out.append(front)
        ln = ptr[front + 1] - ptr[front]
        at = np.repeat(ptr[front] - np.concatenate([[0], np.cumsum(ln)[:-1]]), ln) + np.arange(ln.sum())
        ch = child[at]
        u, cnt = np.unique(ch, return_counts=True)
        left[u] -= cnt
        front = u[left[u] == 0]
    return out


def _solve(col, val, diag, lev, b):
    """x of the triangle: off-diagonals col, val [n][w], diagonal diag [n] (or 1)."""
    x = np.zeros((b.shape[0] + 1, b.shape[1]))
    for r in lev:
        s = b[r].copy()
        for e in range(col.shape[1]):
            s -= val[r, e][:, None] * x[col[r, e]]
        x[r] = s / (diag[r][:, None] if diag is not None else 1.0)
    return x[:-1]


def _fill1(a):
    """A with explicit zeros at its level-1 fill positions."""
    col, _ = _ell(a)
    n, w = col.shape
    i = np.arange(n)
    keys = [np.repeat(i, np.diff(a.rowptr)) * n + a.col]
    for s in range(w):
        k = col[:, s]
        low = k < i
        for u in range(w):
            j = np.where(low, col[np.where(low, k, 0), u], n)
            ok = low & (j < n) & (j > k)
            keys.append(i[ok] * n + j[ok])
    key = np.unique(np.concatenate(keys))
    val = np.zeros(key.size)
    val[np.searchsorted(key, keys[0])] = a.val
    rowptr = np.zeros(n + 1, np.int64)
    np.cumsum(np.bincount(key // n, minlength=n), out=rowptr[1:])
    return SimpleNamespace(n=n, rowptr=rowptr, col=key % n, val=val)


def _factor(a):
    """Incomplete LU over a's pattern: (L off-diagonals, U off-diagonals, U diagonal) and levels."""
    col, val = _ell(a)
    n, w = col.shape
    i = np.arange(n)[:, None]
    dpos = (col < i).sum(axis=1)
    lcol = np.where(col < i, col, n)
    lev = _levels(lcol)
    nlow = int(dpos.max())
    nup = int((col < n).sum(axis=1).max())
    for rows in lev:
        for s in range(nlow):
            r = rows[dpos[rows] > s]
            if not r.size:
                break
            k = col[r, s]
            dk = dpos[k]
            lik = val[r, s] / val[k, dk]
            val[r, s] = lik
            mine = col[r]
            for u in range(1, nup):
                p = dk + u
                has = p < w
                p = np.minimum(p, w - 1)
                j = np.where(has, col[k, p], n)
                if not (j < n).any():
                    break
                hit = (mine == j[:, None]) & (j < n)[:, None]
                val[r] -= hit * (lik * val[k, p])[:, None]
    diag = val[np.arange(n), dpos]
    up = (col > i) & (col < n)
    return lcol, np.where(lcol < n, val, 0.0), np.where(up, col, n), np.where(up, val, 0.0), diag, lev


def _ilu_solve(a, b):
    lcol, lval, ucol, uval, diag, lev = _factor(a)
    return _solve(ucol, uval, diag, _levels(ucol), _solve(lcol, lval, None, lev, b))


def _extended(a, owner, nsub, overlap):
    """Block-diagonal subdomain matrix, its rows' global rows, and which are owned."""
    rows = np.repeat(np.arange(a.n), np.diff(a.rowptr))
    key = owner.astype(np.int64) * a.n + np.arange(a.n)  # (subdomain, row) pairs
    for _ in range(overlap):
        sub, row = key // a.n, key % a.n
        ln = np.diff(a.rowptr)[row]
        at = np.repeat(a.rowptr[row] - np.concatenate([[0], np.cumsum(ln)[:-1]]), ln) + np.arange(ln.sum())
        key = np.unique(np.concatenate([key, np.repeat(sub, ln) * a.n + a.col[at]]))
    key = np.sort(key)
    sub, row = key // a.n, key % a.n
    ln = np.diff(a.rowptr)[row]
    at = np.repeat(a.rowptr[row] - np.concatenate([[0], np.cumsum(ln)[:-1]]), ln) + np.arange(ln.sum())
    want = np.repeat(sub, ln) * a.n + a.col[at]
    pos = np.minimum(np.searchsorted(key, want), key.size - 1)
    ok = key[pos] == want
    er = np.repeat(np.arange(key.size), ln)[ok]
    rowptr = np.zeros(key.size + 1, np.int64)
    np.cumsum(np.bincount(er, minlength=key.size), out=rowptr[1:])
    m = SimpleNamespace(n=key.size, rowptr=rowptr, col=pos[ok], val=a.val[at][ok])
    return m, row, owner[row] == sub


def _poisson_solve(c, b):
    """The Laplacian's solution by sine transforms along each axis."""
    out = b.reshape(c["nz"], c["ny"], c["nx"], -1)
    lam = np.zeros((c["nz"], c["ny"], c["nx"]))
    mats = []
    for ax, d in enumerate((c["nz"], c["ny"], c["nx"])):
        k = np.arange(1, d + 1)
        mats.append(np.sqrt(2.0 / (d + 1)) * np.sin(np.pi * np.outer(k, k) / (d + 1)))
        shape = [1, 1, 1]
        shape[ax] = d
        lam = lam + (2.0 - 2.0 * np.cos(np.pi * k / (d + 1))).reshape(shape)
    for ax, m in enumerate(mats):
        out = np.moveaxis(np.tensordot(m, out, axes=(1, ax)), 0, ax)
    out = out / lam[..., None]
    for ax, m in enumerate(mats):
        out = np.moveaxis(np.tensordot(m, out, axes=(1, ax)), 0, ax)
    return out.reshape(b.shape)


def exact(case, seed):
    c = case
    R = c["nrhs"]
    if c["kind"] == "tri":
        t = _triangle(c, seed)
        b = _rhs_host(t.n, R, seed, c["dtype"])
        col, val = _ell(t)
        i = np.arange(t.n)[:, None]
        low = col < i
        diag = t.val[t.rowptr[1:] - 1]
        lcol = np.where(low, col, t.n)
        return _solve(lcol, np.where(low, val, 0.0), diag, _levels(lcol), b)
    if c["kind"] in ("gmres", "bicgstab"):
        n = c["nx"] * c["ny"] * c["nz"]
        return _poisson_solve(c, _rhs_host(n, R, seed, "f64"))
    if c.get("ilu") == "ilut":
        return None  # rows are dropped one after the other: no vectorised form within the time
    n, off = _neighbours(c)
    grow = 4 if c.get("ilu") == "iluk" else 1
    if n * (R + 6) * grow > 1.6e7:
        return None  # too long in numpy
    if c["kind"] == "batch":
        a, _ = _batch(c, seed)
    else:
        a = _matrix(c, seed)
    b = _rhs_host(a.n, R, seed, "f64")
    if c["kind"] == "sor":
        return _ssor(a, b, c["omega"])
    if c["kind"] == "ras":
        m, row, owned = _extended(a, _owner(c), c["nsub"], c["overlap"])
        z = _ilu_solve(m, b[row])
        out = np.zeros_like(b)
        out[row[owned]] = z[owned]
        return out
    if c.get("ilu") == "iluk":
        a = _fill1(a)
    return _ilu_solve(a, b)


def _rhs_host(n, nrhs, seed, dtype):
    b = np.random.default_rng([seed, 1]).uniform(-1.0, 1.0, (n, nrhs))
    return b.astype(np.float32).astype(np.float64) if dtype == "f32" else b


def _ssor(a, b, omega):
    """A forward, then a backward sweep from x = 0."""
    col, val = _ell(a)
    n = a.n
    i = np.arange(n)[:, None]
    d = val[col == i]
    lcol, ucol = np.where(col < i, col, n), np.where(col > i, col, n)
    lval, uval = np.where(col < i, val, 0.0), np.where((col > i) & (col < n), val, 0.0)

    def times(cc, vv, x):
        xp = np.concatenate([x, np.zeros((1, x.shape[1]))])
        y = np.zeros_like(x)
        for e in range(cc.shape[1]):
            y += vv[:, e][:, None] * xp[cc[:, e]]
        return y

    x = _solve(lcol, lval, d / omega, _levels(lcol), b)
    t = b - times(lcol, lval, x) - (1.0 - 1.0 / omega) * d[:, None] * x
    return _solve(ucol, uval, d / omega, _levels(ucol), t)
