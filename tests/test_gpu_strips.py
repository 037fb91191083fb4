"""The strip form of the self-scheduled solve (triangles whose rows sit on a
regular grid), which the default schedule takes, against the row-wise
schedules bit for bit and against the oracle.

Shapes sit at the edges of the strips: sides of one, just below, at and above
powers of two, chains, thin grids; every stencil; entries dropped from the
stencil; patterns whose offsets look like a grid's but whose entries do not
fit it (those keep the row-wise schedules).
"""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from gpuhelp import bits_equal, dev, dev_tri, host, relerr

pytestmark = pytest.mark.gpu

TOL64, TOL32 = 1e-12, 1e-5


@pytest.fixture(scope="module")
def sp():
    import paper_1710_04985_amd as sp
    assert torch.cuda.is_available()
    return sp


def _dropped(T, seed, keep=0.8):
    """T without a random part of its off-diagonals."""
    rng = np.random.Generator(np.random.PCG64(seed))
    rows = np.repeat(np.arange(T.n), np.diff(T.row_ptr))
    k = (T.col_idx == rows) | (rng.random(T.nnz) < keep)
    rp = np.zeros(T.n + 1, np.int64)
    np.cumsum(np.bincount(rows[k], minlength=T.n), out=rp[1:])
    return W.Triangle(T.n, rp.astype(np.int32), T.col_idx[k], T.vals[k], T.upper, T.unit_diag,
                      T.name + "_dropped")


def _banded(n, offsets, upper=False):
    """Every entry at the given offsets that fits in the matrix (wraps around
    the lines of any grid)."""
    i = np.arange(n)
    cols, vals, rp = [], [], [0]
    for r in range(n):
        c = sorted(j for j in ([r + o for o in offsets] if upper else [r - o for o in offsets])
                   if 0 <= j < n)
        c = [r] + c if upper else c + [r]
        cols += c
        vals += [float(len(offsets) + 1) if j == r else -1.0 for j in c]
        rp.append(len(cols))
    return W.Triangle(n, np.array(rp, np.int32), np.array(cols, np.int32), np.array(vals),
                      upper=upper, name="band%s" % "_".join(map(str, offsets)))


def _varied(T, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    rows = np.repeat(np.arange(T.n), np.diff(T.row_ptr))
    T.vals = np.where(T.col_idx == rows, T.vals * rng.uniform(0.8, 1.3, T.nnz),
                      T.vals * rng.uniform(-1.0, 1.0, T.nnz))
    return T


GRIDS = [((1, 1), 5), ((2, 3), 5), ((3, 3), 9), ((64, 64), 5), ((65, 63), 5), ((63, 130), 9),
         ((200, 7), 9), ((5, 300), 9), ((8, 8, 8), 7), ((9, 7, 5), 7), ((33, 20, 17), 7),
         ((70, 3, 40), 7), ((2, 2, 50), 7), ((12, 11, 13), 27), ((4, 33, 6), 27), ((40, 5, 9), 27)]


@pytest.mark.parametrize("setup", ["host", "device"])
@pytest.mark.parametrize("upper", [False, True])
@pytest.mark.parametrize("dims,points", GRIDS, ids=["x".join(map(str, g)) + "_%d" % p for g, p in GRIDS])
def test_grid_equals_row_wise_bitwise(sp, dims, points, upper, setup):
    o = oracle.get()
    for T in (_varied(W.stencil_triangle(dims, points, upper=upper), 3),
              _dropped(_varied(W.stencil_triangle(dims, points, upper=upper), 4), 5)):
        for dt, tol in ((torch.float64, TOL64), (torch.float32, TOL32)):
            d = dev_tri(T, dt)
            uplo = "U" if upper else "L"
            b = dev(W.uniform_vector(T.n, 5), dt)
            h = sp.Handle(*d, uplo=uplo, setup=setup).configure(algo=2)
            ref = sp.Handle(*d, uplo=uplo, setup=setup).configure(algo=2, assign=0)
            for _ in range(3):
                x, y = h.solve(b), h.solve_t(b)
                h.status()
                assert bits_equal(x, ref.solve(b)) and bits_equal(y, ref.solve_t(b))
            v = host(d[2]).astype(np.float64)
            xo = o.solve(T.row_ptr, T.col_idx, v, host(b).astype(np.float64), upper)
            assert relerr(host(x), xo) <= tol


PATTERNS = [W.bidiagonal_fast(1000, 2.0, 1.0), W.bidiagonal_fast(777, 2.0, 1.0, upper=True),
            W.diagonal_matrix(np.linspace(1, 2, 500)), _banded(900, [1, 30]),
            _banded(900, [30, 31]), _banded(900, [29, 30]), _banded(1000, [1, 10, 100], upper=True),
            _banded(700, [3, 17]), _banded(640, [2, 4, 8, 16])]


@pytest.mark.parametrize("T", PATTERNS, ids=[t.name + ("U" if t.upper else "L") for t in PATTERNS])
def test_other_offset_patterns(sp, T):
    """Chains, independent rows, and bands that run across the line ends of
    the grid their offsets suggest."""
    o = oracle.get()
    b = W.uniform_vector(T.n, 6)
    uplo = "U" if T.upper else "L"
    h = sp.Handle(*dev_tri(T), uplo=uplo).configure(algo=2)
    ref = sp.Handle(*dev_tri(T), uplo=uplo).configure(algo=2, assign=0)
    x, y = h.solve(dev(b)), h.solve_t(dev(b))
    h.status()
    assert bits_equal(x, ref.solve(dev(b))) and bits_equal(y, ref.solve_t(dev(b)))
    assert relerr(host(x), o.solve(T.row_ptr, T.col_idx, T.vals, b, T.upper)) <= TOL64


def test_batched_grids(sp):
    """Systems of different grids in one handle, an empty and a one-row system
    among them; with a system that is no grid, the whole handle is row-wise."""
    tris = [W.ilu0_lower((s, t)) for s, t in ((7, 9), (33, 20), (64, 64), (5, 70))]
    tris += [W.laplacian_triangle((6, 5, 4)), W.diagonal_matrix(np.array([2.0])),
             W.stencil_triangle((9, 10), 9)]
    empty = W.Triangle(0, np.zeros(1, np.int32), np.zeros(0, np.int32), np.zeros(0))
    for sys in (tris, tris[:2] + [empty] + tris[2:], tris + [_banded(300, [2, 5, 7])]):
        devs = [dev_tri(t) for t in sys]
        b = dev(W.uniform_vector(sum(t.n for t in sys), 8))
        mk = lambda **o: sp.BatchedHandle([d[0] for d in devs], [d[1] for d in devs],
                                          [d[2] for d in devs]).configure(**o)
        h, ref = mk(algo=2), mk(algo=2, assign=0)
        for _ in range(3):
            assert bits_equal(h.solve(b), ref.solve(b)) and bits_equal(h.solve_t(b), ref.solve_t(b))
        h.status()


def test_special_values(sp):
    """Infinities, NaN and products that underflow to signed zeros give the
    bits of the row-wise schedules (NaN in the same places), and stay in the
    rows that depend on them."""
    for T in (W.laplacian_triangle((40, 30)), W.stencil_triangle((11, 10, 9), 27),
              _dropped(W.laplacian_triangle((14, 13, 12)), 2)):
        b = W.uniform_vector(T.n, 31)
        rows = np.repeat(np.arange(T.n), np.diff(T.row_ptr))
        b[T.n // 2] = np.inf
        b[T.n // 3] = np.nan
        tiny = np.where(T.col_idx == rows, 1.0, T.vals * 1e-200)
        bt = W.uniform_vector(T.n, 32) * 1e-200
        bt[::7] = -0.0
        for v, bb in ((T.vals, b), (tiny, bt)):
            d = (dev(T.row_ptr), dev(T.col_idx), dev(v))
            x = host(sp.Handle(*d).configure(algo=2).solve(dev(bb)))
            r = host(sp.Handle(*d).configure(algo=2, assign=0).solve(dev(bb)))
            assert np.array_equal(np.isnan(x), np.isnan(r))
            ok = ~np.isnan(r)
            assert bits_equal(x[ok], r[ok])


def test_unit_diagonal_update_in_place_and_graph(sp):
    T = W.laplacian_triangle((31, 17, 12))
    T.unit_diag = True
    d = dev_tri(T)
    b = dev(W.uniform_vector(T.n, 9))
    h = sp.Handle(*d, unit_diag=True).configure(algo=2)
    ref = sp.Handle(*d, unit_diag=True).configure(algo=2, assign=0)
    x = b.clone()
    h.solve(x, out=x)
    assert bits_equal(x, ref.solve(b))
    h.prepare_transpose()
    v2 = dev(T.vals * np.linspace(0.1, 0.3, T.nnz))
    h.update_values(v2)
    ref.update_values(v2)
    assert bits_equal(h.solve(b), ref.solve(b)) and bits_equal(h.solve_t(b), ref.solve_t(b))
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        y = torch.empty_like(b)
        g, gt = h.capture(b, y, stream=s), h.capture(b, y, transpose=True, stream=s)
        for k in range(4):
            g.launch(s)
            s.synchronize()
            assert bits_equal(y, ref.solve(b))
            h.solve(b * 2.0)
            gt.launch(s)
            s.synchronize()
            assert bits_equal(y, ref.solve_t(b))
            v3 = v2 * (1.0 + k)            # a graph reads the handle's current values
            h.update_values(v3)
            ref.update_values(v3)
    h.status()


@pytest.mark.parametrize("coop", [0, 1])
def test_watchdog_and_residency(sp, coop):
    """Waits that give up (forced from the host) drain, are reported, and the
    handle then works; a grid needs no residency (strips come from a ticket),
    so the residency limit changes nothing."""
    T = W.laplacian_triangle((40, 41, 42))
    b = dev(W.uniform_vector(T.n, 10))
    ref = sp.Handle(*dev_tri(T)).configure(algo=2, assign=0).solve(b)
    h = sp.Handle(*dev_tri(T)).configure(algo=2, cooperative=coop)
    h.set_option("spin_limit", 1)
    h.solve(b)
    with pytest.raises(sp.SpTRSVError) as e:
        h.status()
    assert e.value.status == -10
    h.configure(spin_limit=1 << 22, residency_limit=0)
    for _ in range(3):
        assert bits_equal(h.solve(b), ref)
    h.status()


@pytest.mark.parametrize("nrhs", [2, 3, 16, 33])
@pytest.mark.parametrize("dims,points", [((65, 40), 5), ((40, 33), 9), ((17, 9, 20), 7), ((9, 8, 10), 27)])
def test_several_right_hand_sides(sp, dims, points, nrhs):
    """Every column equals the one-lane-per-row solve bit for bit, plain and
    transposed, with a column stride beyond n and in place."""
    T = _varied(W.stencil_triangle(dims, points), 6)
    for dt in (torch.float64, torch.float32):
        d = dev_tri(T, dt)
        wide = torch.zeros(nrhs, T.n + 7, dtype=dt, device="cuda:0")
        for r in range(nrhs):
            wide[r, :T.n] = dev(W.uniform_vector(T.n, 40 + r), dt)
        B = wide[:, :T.n]
        h = sp.Handle(*d).configure(algo=2)
        one = sp.Handle(*d).configure(algo=1, group=1)
        for tr in (False, True):
            X = h.solve_multi(B, transpose=tr)
            h.status()
            for r in range(nrhs):
                b = B[r].contiguous()
                assert bits_equal(X[r].contiguous(), one.solve_t(b) if tr else one.solve(b)), (tr, r)
        ref = h.solve_multi(B)
        h.solve_multi(B, out=B)
        h.status()
        assert bits_equal(B.contiguous(), ref.contiguous())
        assert not wide[:, T.n:].any()                 # nothing written past the columns


@pytest.mark.parametrize("upper", [False, True])
def test_levels_of_device_setup(sp, upper):
    """Levels read off the grid, or found by the sweep where rows lack entries
    or wrap around the lines, equal the host's; also of a batch."""
    tris = [W.stencil_triangle(d, p, upper=upper) for d, p in GRIDS]
    tris += [_dropped(t, 7) for t in tris[4:]] + [t for t in PATTERNS if t.upper == upper]
    uplo = "U" if upper else "L"
    for T in tris:
        devh, hosth = (sp.Handle(*dev_tri(T), uplo=uplo, setup=s) for s in ("device", "host"))
        for tr in (False, True):
            for a, b in zip(devh.export_analysis(tr), hosth.export_analysis(tr)):
                assert np.array_equal(a, b)
    for part in (tris[:12], tris[:20]):
        d = [dev_tri(t) for t in part]
        devh, hosth = (sp.BatchedHandle([a[0] for a in d], [a[1] for a in d], [a[2] for a in d],
                                        uplo=uplo, setup=s) for s in ("device", "host"))
        for a, b in zip(devh.export_analysis(), hosth.export_analysis()):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("nrhs", [1, 3])
def test_long_records_loaded_further_ahead(sp, nrhs):
    """13 entries a row in FP64, on both sides of the 64 MB of records from
    which they are loaded further ahead (about 20 and 110 MB)."""
    for side in (45, 80):
        T = _varied(W.stencil_triangle((side, side, side), 27), 6)
        d = dev_tri(T)
        b = torch.stack([dev(W.uniform_vector(T.n, 20 + q)) for q in range(nrhs)])
        h = sp.Handle(*d, setup="device").configure(algo=2)
        ref = sp.Handle(*d, setup="device").configure(algo=2, assign=0, **({"group": 1} if nrhs > 1 else {}))
        for _ in range(2):
            x = h.solve_multi(b) if nrhs > 1 else h.solve(b[0])[None]
            h.status()
            for q in range(nrhs):
                assert bits_equal(x[q], ref.solve(b[q]))
