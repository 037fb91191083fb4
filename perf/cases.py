"""The solves, set-ups and gradients that users of this library run, as timed cases.

A case names a pattern, its size, the value type and the call:

  lu       the lower and then the upper solve of one grid operator, y = U^-1 (L^-1 b):
           the application of a preconditioner, and the paper's own experiment
  solve    one triangle, one right-hand side (plain or transposed)
  batch    independent factors of different sizes, solved by one call
  multi    several right-hand sides of one triangle (plain or transposed)
  adjoint  forward solve and gradients with respect to values and right-hand side
  setup    analysis of a new pattern on the device, and its first solve

Patterns: "grid" (triangles of the 5-, 7-, 9- or 27-point operator on nx x ny (x nz),
natural order), "ilu" (unit-lower ILU(0) factor of the 5- or 7-point operator) and
"power" (random rows whose lengths follow a power law on [1, 2000], mean 8, columns
within 50,000 of the diagonal: the stand-in for general matrices).
"""
import math
import random

import torch

import paper_1710_04985_amd as sp

DEV = "cuda:0"
TYPES = {"f64": torch.float64, "f32": torch.float32}
ALPHA, KMAX, WINDOW = 1.85508818062782, 2000, 50000


def listed():
    return [
        # the smallest call: a 2-D problem of 4,096 unknowns, where launches and latency count
        {"name": "grid2d_64_solve", "kind": "solve", "pattern": "grid", "points": 5, "nx": 64, "ny": 64, "nz": 1, "dtype": "f64"},
        # the benchmark's step: both triangles of the 3-D 7-point operator, two million unknowns
        {"name": "grid3d_128_lu", "kind": "lu", "pattern": "grid", "points": 7, "nx": 128, "ny": 128, "nz": 128, "dtype": "f64"},
        # the same step in single precision on a grid whose sides divide by nothing
        {"name": "grid3d_odd_lu_f32", "kind": "lu", "pattern": "grid", "points": 7, "nx": 61, "ny": 83, "nz": 47, "dtype": "f32"},
        # a deep 2-D problem: four short entries a row, 3,070 levels
        {"name": "grid2d_9pt_1024_lu", "kind": "lu", "pattern": "grid", "points": 9, "nx": 1024, "ny": 1024, "nz": 1, "dtype": "f64"},
        # a wide stencil: thirteen entries a row, the most bytes of the single solves
        {"name": "grid3d_27pt_128_lu", "kind": "lu", "pattern": "grid", "points": 27, "nx": 128, "ny": 128, "nz": 128, "dtype": "f64"},
        # a general matrix: irregular levels, rows up to 2,000 entries
        {"name": "power_1m_solve", "kind": "solve", "pattern": "power", "n": 1000000, "dtype": "f64", "trans": False},
        # the transposed solve of the same family in single precision, an odd size
        {"name": "power_777k_solve_t_f32", "kind": "solve", "pattern": "power", "n": 777777, "dtype": "f32", "trans": True},
        # 256 small factors of different sizes in one call
        {"name": "batch_256_ilu2d", "kind": "batch", "count": 256, "lo": 32, "hi": 256, "pick": 4, "dtype": "f64"},
        # block methods: sixteen right-hand sides at once
        {"name": "grid3d_128_rhs16", "kind": "multi", "pattern": "grid", "points": 7, "nx": 128, "ny": 128, "nz": 128, "dtype": "f64", "nrhs": 16, "trans": False},
        # a few right-hand sides, transposed, single precision
        {"name": "ilu3d_96_rhs3_t_f32", "kind": "multi", "pattern": "ilu", "nx": 96, "ny": 96, "nz": 96, "dtype": "f32", "nrhs": 3, "trans": True},
        # training through a solve: new values, forward, both gradients
        {"name": "ilu3d_96_adjoint", "kind": "adjoint", "pattern": "ilu", "nx": 96, "ny": 96, "nz": 96, "dtype": "f64"},
        # a new pattern: analysis on the device and the first solve
        {"name": "grid3d_128_setup", "kind": "setup", "pattern": "grid", "points": 7, "nx": 128, "ny": 128, "nz": 128, "dtype": "f64"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _grid_dims(rng, d3, most):
    if d3:
        while True:
            nx, ny, nz = (_log(rng, 9, 128) for _ in range(3))
            if nx * ny * nz <= most:
                return nx, ny, nz
    nx, ny = (_log(rng, 31, 1024) for _ in range(2))
    return nx, max(2, min(ny, most // nx)), 1


def draw(rng):
    kind = rng.choice(["lu", "lu", "solve", "batch", "multi", "adjoint", "setup"])
    c = {"kind": kind, "dtype": rng.choice(["f64", "f64", "f32"])}
    if kind == "batch":
        lo = rng.randint(16, 96)
        c.update(count=_log(rng, 4, 256), lo=lo, hi=rng.randint(lo, 255), pick=rng.randint(0, 1 << 20))
        return c
    if kind in ("solve", "multi", "adjoint"):
        c["trans"] = rng.random() < 0.4
    if kind == "multi":
        c["nrhs"] = rng.randint(2, 16)
    if kind == "adjoint":
        del c["trans"]
    # unknowns (times right-hand sides) up to the largest listed case
    most = (1 << 21) if kind != "multi" else min(1 << 21, (1 << 25) // c["nrhs"])
    which = rng.choice(["grid", "grid", "ilu", "power"])
    if kind == "lu":
        which = "grid"
    elif kind == "adjoint":
        which = "ilu"
    if which == "power":
        c.update(pattern="power", n=_log(rng, 10000, 300000 if kind in ("setup", "multi") else 1000000))
        return c
    d3 = rng.random() < 0.6
    nx, ny, nz = _grid_dims(rng, d3, most)
    c.update(pattern=which, nx=nx, ny=ny, nz=nz)
    if which == "grid":
        c["points"] = rng.choice([7, 7, 27] if d3 else [5, 9])
        if kind in ("multi", "setup"):
            c["points"] = 7 if d3 else 5
    return c


# ------------------------------------------------------------------ inputs

def _offsets(points, d3):
    if points in (5, 7):
        return [(-1, 0, 0), (0, -1, 0)] + ([(0, 0, -1)] if d3 else [])
    zs = (-1, 0) if d3 else (0,)
    return [(x, y, z) for z in zs for y in (-1, 0, 1) for x in (-1, 0, 1) if (z, y, x) < (0, 0, 0)]


def _grid(nx, ny, nz, points, upper=False):
    """row_ptr, col_idx and the off-diagonal mask of one triangle, columns ascending."""
    d3 = nz > 1 or points in (7, 27)
    n = nx * ny * nz
    i = torch.arange(n, device=DEV, dtype=torch.int64)
    x, y, z = i % nx, (i // nx) % ny, i // (nx * ny)
    sign = -1 if upper else 1
    offs = sorted((sign * (a + nx * b + nx * ny * c), sign * a, sign * b, sign * c) for a, b, c in _offsets(points, d3))
    offs = offs + [(0, 0, 0, 0)] if not upper else [(0, 0, 0, 0)] + offs
    keep, cols = [], []
    for lin, a, b, c in offs:
        ok = (x + a >= 0) & (x + a < nx) & (y + b >= 0) & (y + b < ny) & (z + c >= 0) & (z + c < nz)
        keep.append(ok)
        cols.append((i + lin).to(torch.int32))
    keep = torch.stack(keep, 1)
    col = torch.stack(cols, 1)[keep]
    rp = torch.zeros(n + 1, device=DEV, dtype=torch.int64)
    rp[1:] = keep.sum(1).cumsum(0)
    return rp, col


def _rows(rp):
    return torch.repeat_interleave(torch.arange(rp.numel() - 1, device=DEV), rp[1:] - rp[:-1])


def _pivots(nx, ny, nz, d3):
    """Pivots of ILU(0): d = c - sum of 1/d over the lower grid neighbours, as a fixed point."""
    d = torch.full((nz, ny, nx), 6.0 if d3 else 4.0, device=DEV, dtype=torch.float64)
    for k in range(nx + ny + nz):
        e = torch.full_like(d, 6.0 if d3 else 4.0)
        e[:, :, 1:] -= 1.0 / d[:, :, :-1]
        e[:, 1:, :] -= 1.0 / d[:, :-1, :]
        e[1:, :, :] -= 1.0 / d[:-1, :, :]
        if k % 16 == 15 and torch.equal(d, e):
            break
        d = e
    return d


def _ilu(nx, ny, nz, piv=None):
    d3 = nz > 1
    rp, col = _grid(nx, ny, nz, 7 if d3 else 5)
    piv = _pivots(nx, ny, nz, d3) if piv is None else piv[:nz, :ny, :nx]
    v = -1.0 / piv.reshape(-1)[col.long()]
    v[(rp[1:] - 1)] = 1.0
    return rp, col, v


def _power(n, gen):
    k = torch.arange(1, KMAX + 1, device=DEV, dtype=torch.float64) ** -ALPHA
    cdf = torch.cumsum(k, 0) / k.sum()
    i = torch.arange(n, device=DEV, dtype=torch.int64)
    lo = (i - WINDOW).clamp(min=0)
    u = torch.rand(n, device=DEV, dtype=torch.float64, generator=gen)
    cnt = torch.minimum(torch.searchsorted(cdf, u).clamp(max=KMAX - 1) + 1, i - lo)
    row = torch.repeat_interleave(i, cnt)
    span = (row - lo[row])
    u = torch.rand(row.numel(), device=DEV, dtype=torch.float64, generator=gen)
    col = lo[row] + torch.minimum((u * span).long(), span - 1)
    key = torch.unique(torch.cat([row * n + col, i * n + i]))
    row, col = key // n, key % n
    cnt = torch.bincount(row, minlength=n)
    rp = torch.zeros(n + 1, device=DEV, dtype=torch.int64)
    rp[1:] = cnt.cumsum(0)
    v = (2 * torch.rand(row.numel(), device=DEV, dtype=torch.float64, generator=gen) - 1) / (cnt[row] - 1).clamp(min=1)
    v[rp[1:] - 1] = 1 + torch.rand(n, device=DEV, dtype=torch.float64, generator=gen)
    return rp, col.to(torch.int32), v


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _uniform(shape, gen, dt):
    return (2 * torch.rand(shape, device=DEV, dtype=torch.float64, generator=gen) - 1).to(dt)


def _triangle(c, gen, upper=False):
    """(row_ptr int32, col_idx int32, values) of the case's triangle."""
    dt = TYPES[c["dtype"]]
    if c["pattern"] == "power":
        rp, col, v = _power(c["n"], gen)
    elif c["pattern"] == "ilu":
        rp, col, v = _ilu(c["nx"], c["ny"], c["nz"])
    else:
        rp, col = _grid(c["nx"], c["ny"], c["nz"], c["points"], upper)
        # the stencils' diagonals: the number of neighbours
        v = torch.full((col.numel(),), -1.0, device=DEV, dtype=torch.float64)
        v[(rp[:-1] if upper else rp[1:] - 1)] = float(c["points"] - 1)
    return rp.to(torch.int32), col, v.to(dt)


def _sides(c):
    r = random.Random(c["pick"])
    return [r.randint(c["lo"], c["hi"]) for _ in range(c["count"])]


def _batch(c):
    piv = _pivots(c["hi"], c["hi"], 1, False)
    made = {}
    for s in _sides(c):
        if s not in made:
            rp, col, v = _ilu(s, s, 1, piv)
            made[s] = (rp.to(torch.int32), col, v.to(TYPES[c["dtype"]]))
    return [made[s] for s in _sides(c)]


def _inputs(c, seed):
    gen, dt = _gen(seed), TYPES[c["dtype"]]
    if c["kind"] == "batch":
        tris = _batch(c)
        return {"tris": tris, "b": _uniform(sum(t[0].numel() - 1 for t in tris), gen, dt)}
    s = {"tri": _triangle(c, gen)}
    n = s["tri"][0].numel() - 1
    if c["kind"] == "lu":
        s["tri_u"] = _triangle(c, gen, upper=True)
    s["b"] = _uniform((c["nrhs"], n) if c["kind"] == "multi" else n, gen, dt)
    if c["kind"] == "adjoint":
        s["w"] = _uniform(n, gen, dt)
    return s


def prepare(c, seed):
    s = _inputs(c, seed)
    s["kind"], s["trans"] = c["kind"], bool(c.get("trans"))
    if c["kind"] == "batch":
        t = s["tris"]
        s["h"] = sp.BatchedHandle([a[0] for a in t], [a[1] for a in t], [a[2] for a in t], setup="device")
    elif c["kind"] != "setup":
        s["h"] = sp.Handle(*s["tri"], uplo="L", setup="device")
    if c["kind"] == "lu":
        s["hu"] = sp.Handle(*s["tri_u"], uplo="U", setup="device")
    if s["trans"] or c["kind"] == "adjoint":
        s["h"].prepare_transpose()
    if c["kind"] == "adjoint":
        s["vals"] = s["tri"][2].clone().requires_grad_(True)
        s["b"].requires_grad_(True)
    return s


def run(s):
    k, b = s["kind"], s["b"]
    if k == "lu":
        y = s["h"].solve(b)
        return y, s["hu"].solve(y)
    if k == "solve":
        return s["h"].solve_t(b) if s["trans"] else s["h"].solve(b)
    if k == "batch":
        return s["h"].solve(b)
    if k == "multi":
        return s["h"].solve_multi(b, transpose=s["trans"])
    if k == "adjoint":
        x = sp.sptrsv(s["vals"], b, s["h"])
        gv, gb = torch.autograd.grad(x, (s["vals"], b), s["w"])
        return x.detach(), gv, gb
    h = sp.Handle(*s["tri"], uplo="L", setup="device")
    return h.solve(b)


def _size(c):
    """(unknowns, stored off-diagonals) of one triangle; the power-law count is the mean."""
    if c["kind"] == "batch":
        return sum(s * s for s in _sides(c)), sum(2 * s * (s - 1) for s in _sides(c))
    if c["pattern"] == "power":
        return c["n"], 8 * c["n"]
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    points = c.get("points", 7 if nz > 1 else 5)
    offs = _offsets(points, nz > 1 or points in (7, 27))
    return nx * ny * nz, sum((nx - abs(a)) * (ny - abs(b)) * (nz - abs(d)) for a, b, d in offs)


def work(c):
    n, off = _size(c)
    vb = 8 if c["dtype"] == "f64" else 4
    k = c.get("nrhs", 1)
    matrix = (off + n) * (vb + 4) + 4 * (n + 1)
    solve = matrix + 2 * k * n * vb
    flops = k * 2 * (off + n)
    if c["kind"] == "lu":
        return {"bytes": 2 * solve, "flops": 2 * flops}
    if c["kind"] == "adjoint":
        # both solves, the new values read, the gradient of the values written
        return {"bytes": 2 * solve + 2 * (off + n) * vb, "flops": 2 * flops + off + n}
    return {"bytes": solve, "flops": flops}


# ------------------------------------------------- the same in 64 bits

def _substitute(rp, col, v, b):
    """T x = b by x <- (b - N x) / d, d the diagonal and N the rest of T, repeated until
    nothing changes: N is nilpotent, so this ends at substitution's own result."""
    row, col = _rows(rp.long()), col.long()
    off = row != col
    d = torch.ones_like(b)
    d[row[~off]] = v[~off]
    cnt = torch.bincount(row[off], minlength=b.numel())
    ptr = torch.zeros(b.numel() + 1, device=DEV, dtype=torch.int64)
    ptr[1:] = cnt.cumsum(0)
    c, w = col[off], v[off]
    x = b / d
    for k in range(b.numel() + 1):
        s = torch.segment_reduce(w * x[c], "sum", offsets=ptr, initial=0.0, unsafe=True)
        y = (b - s) / d
        if k % 8 == 7 and torch.equal(x, y):
            break
        x = y
    return x


def _transposed(rp, col, v):
    row = _rows(rp.long())
    order = torch.argsort(col.long() * (rp.numel() - 1) + row)
    ptr = torch.zeros_like(rp)
    ptr[1:] = torch.bincount(col.long(), minlength=rp.numel() - 1).cumsum(0)
    return ptr, row[order], v[order]


def exact(c, seed):
    s = _inputs(c, seed)
    b = s["b"].double()
    if c["kind"] == "batch":
        at, rps, cols, vals = 0, [], [], []
        base = 0
        for rp, col, v in s["tris"]:
            rps.append(rp[:-1].long() + base)
            cols.append(col.long() + at)
            vals.append(v.double())
            at += rp.numel() - 1
            base += col.numel()
        rps.append(torch.tensor([base], device=DEV))
        return _substitute(torch.cat(rps), torch.cat(cols), torch.cat(vals), b)
    rp, col, v = s["tri"][0], s["tri"][1], s["tri"][2].double()
    if c["kind"] == "lu":
        y = _substitute(rp, col, v, b)
        rp, col, v = s["tri_u"]
        return y, _substitute(rp, col, v.double(), y)
    if c["kind"] == "adjoint":
        x = _substitute(rp, col, v, b)
        gb = _substitute(*_transposed(rp, col, v), s["w"].double())
        return x, -gb[_rows(rp.long())] * x[col.long()], gb
    if c.get("trans"):
        rp, col, v = _transposed(rp, col, v)
    if c["kind"] == "multi":
        return torch.stack([_substitute(rp, col, v, b[q]) for q in range(c["nrhs"])])
    return _substitute(rp, col, v, b)
