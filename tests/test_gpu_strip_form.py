"""Which form a solve takes, as the library reports it: strips on grids, the
row-wise schedules elsewhere and wherever an option asks for them."""
import numpy as np
import pytest
import torch

import workloads as W
from gpuhelp import bits_equal, dev, dev_tri
from test_gpu_strips import GRIDS, _banded, _dropped
from test_strips_cpu import band

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sp():
    import paper_1710_04985_amd as sp
    assert torch.cuda.is_available()
    return sp


@pytest.mark.parametrize("setup", ["host", "device"])
@pytest.mark.parametrize("dims,points", GRIDS, ids=["x".join(map(str, g)) + "_%d" % p for g, p in GRIDS])
def test_grids_take_strips(sp, dims, points, setup):
    for upper in (False, True):
        T = W.stencil_triangle(dims, points, upper=upper)
        for t in (T, _dropped(T, 5)):
            for dt in (torch.float64, torch.float32):
                h = sp.Handle(*dev_tri(t, dt), uplo="U" if upper else "L", setup=setup).configure(algo=2)
                assert h.strips(transpose=True)["strips"] == 0      # not analysed yet
                h.prepare_transpose()
                for tr in (False, True):
                    rows = np.bincount(t.col_idx) if tr else np.diff(t.row_ptr)
                    longest = max(rows.max() - 1, 2)
                    for nrhs in (1, 3, 16):
                        s = h.strips(nrhs, tr)
                        assert s["strips"] > 0
                        assert s["slots"] == longest if longest <= 4 else s["slots"] in (13, 15)
                        assert s["sums"] == (4 if longest > 4 and nrhs == 1 else 1)
                        assert s["depth"] == (16 if longest <= 4 else 8 if dt == torch.float32 else 4)
                for o in ({"assign": 0}, {"algo": 1}, {"group": 1}, {"wg": 128}, {"poll": 0}):
                    g = sp.Handle(*dev_tri(t, dt), uplo="U" if upper else "L", setup=setup)
                    assert g.configure(**{"algo": 2, **o}).strips()["strips"] == 0


def test_what_is_no_grid_stays_row_wise(sp):
    """Bands that run across the line ends of the grid their offsets suggest,
    an irregular triangle, and a batch with one system that is no grid."""
    for T in (_banded(900, [1, 30]), _banded(900, [29, 30]), _banded(1000, [1, 10, 100], upper=True),
              _banded(900, [2, 5, 7]), W.powerlaw_lower(5000, 3, window=700)):
        h = sp.Handle(*dev_tri(T), uplo="U" if T.upper else "L").configure(algo=2)
        h.prepare_transpose()
        assert h.strips()["strips"] == 0 and h.strips(transpose=True)["strips"] == 0
    grids = [W.ilu0_lower((s, t)) for s, t in ((33, 20), (64, 64), (25, 70))]
    for tris, want in ((grids, True), (grids + [_banded(300, [2, 5, 7])], False)):
        d = [dev_tri(t) for t in tris]
        h = sp.BatchedHandle([a[0] for a in d], [a[1] for a in d], [a[2] for a in d]).configure(algo=2)
        h.prepare_transpose()
        assert (h.strips()["strips"] > 0) == want and (h.strips(transpose=True)["strips"] > 0) == want


def test_both_depths_of_long_fp64_records(sp):
    """Records of 13 entries a row on both sides of the size from which they
    are loaded further ahead, against the row-wise schedule bit for bit."""
    for side, depth, several in ((45, 4, 4), (72, 4, 4), (80, 4, 8), (90, 8, 8)):
        T = W.stencil_triangle((side, side, side), 27)
        d, b = dev_tri(T), dev(W.uniform_vector(T.n, 20))
        h = sp.Handle(*d, setup="device")
        assert h.strips()["depth"] == depth and h.strips(2)["depth"] == several
        x = h.solve(b)
        h.status()
        assert bits_equal(x, sp.Handle(*d, setup="device").configure(algo=2, assign=0).solve(b))


@pytest.mark.parametrize("n,offsets", [(7000, [1000]), (17321, [1000]), (100000, [5000]), (4096, [64, 1024]),
                                       (4001, [64, 1024]), (6000, [1, 600])])
@pytest.mark.parametrize("setup", ["host", "device"])
def test_lines_without_coupling(sp, n, offsets, setup):
    """Entries one line or plane back only: strips whose lanes, or which
    themselves, do not depend on one another, against the row-wise schedule."""
    T = band(n, offsets)
    T.vals = np.where(T.col_idx == np.repeat(np.arange(n), np.diff(T.row_ptr)), 1.5,
                      np.random.default_rng(3).uniform(-1, 1, T.nnz))
    for dt in (torch.float64, torch.float32):
        d, b = dev_tri(T, dt), dev(W.uniform_vector(n, 7), dt)
        h = sp.Handle(*d, setup=setup).configure(algo=2)
        h.prepare_transpose()
        assert h.strips()["strips"] and h.strips(transpose=True)["strips"] and h.strips(3)["strips"]
        ref = sp.Handle(*d, setup=setup).configure(algo=2, assign=0)
        for _ in range(2):
            assert bits_equal(h.solve(b), ref.solve(b)) and bits_equal(h.solve_t(b), ref.solve_t(b))
        X = h.solve_multi(torch.stack([b, 2 * b, -b]))
        assert bits_equal(X[1], ref.solve(2 * b)) and bits_equal(X[2], ref.solve(-b))
        h.status()


@pytest.mark.parametrize("setup", ["host", "device"])
def test_shallow_triangles_are_solved_row_wise(sp, setup):
    """Far fewer levels than a line of the grid has rows."""
    chains = band(16384, [1])
    cut = (chains.col_idx % 256 != 255) | (chains.col_idx == np.repeat(np.arange(16384), np.diff(chains.row_ptr)))
    rp = np.concatenate([[0], np.cumsum(np.add.reduceat(cut, chains.row_ptr[:-1]))]).astype(np.int32)
    for T in (band(20000, []), band(400000, [100000]),
              W.Triangle(16384, rp, chains.col_idx[cut], chains.vals[cut])):
        d, b = dev_tri(T), dev(W.uniform_vector(T.n, 7))
        h = sp.Handle(*d, setup=setup)
        h.prepare_transpose()
        assert not any(h.strips(k, t)["strips"] for k in (1, 8) for t in (False, True))
        x, one = h.solve(b), sp.Handle(*d, setup=setup).configure(algo=1, group=1)
        h.status()
        assert bits_equal(x, one.solve(b)) and bits_equal(h.solve_t(b), one.solve_t(b))


def test_set_up_of_small_systems_beside_a_long_chain(sp):
    """5000 systems of 16x16 and a chain of 125,000 rows: the construction's work
    follows the records, not the systems times the longest one's steps."""
    small, chain = W.laplacian_triangle((16, 16)), W.bidiagonal_fast(125000, 2.0, 1.0)
    ds, dc = dev_tri(small), dev_tri(chain)
    d = [ds] * 5000 + [dc]
    b = dev(W.uniform_vector(5000 * 256 + chain.n, 3))
    one, long = sp.Handle(*ds).configure(algo=2, assign=0), sp.Handle(*dc).configure(algo=2, assign=0)
    times = []
    for _ in range(3):
        h = sp.BatchedHandle([a[0] for a in d], [a[1] for a in d], [a[2] for a in d], setup="device")
        assert h.strips()["strips"] == 5001
        times.append(h.setup_info()[1])
    x = h.solve(b)
    h.status()
    for k in (0, 2500, 4999):
        assert bits_equal(x[256 * k:256 * (k + 1)], one.solve(b[256 * k:256 * (k + 1)].clone()))
    assert bits_equal(x[5000 * 256:], long.solve(b[5000 * 256:].clone()))
    assert min(times) < 20, times                        # measured 12; 41 before


def test_values_updated_while_another_form_is_chosen(sp):
    """A solve in strips after updates that ran under another form, eagerly and
    from a graph, reads the newest values."""
    T = W.laplacian_triangle((31, 17, 12))
    d, b = dev_tri(T), dev(W.uniform_vector(T.n, 9))
    h, ref = sp.Handle(*d), sp.Handle(*d).configure(algo=2, assign=0)
    h.prepare_transpose()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        y = torch.empty_like(b)
        for k in range(3):
            v = d[2] * (1.0 + 0.25 * k)
            h.configure(algo=1)
            h.update_values(v)
            ref.update_values(v)
            assert bits_equal(h.solve(b), ref.solve(b))
            h.configure(algo=0)
            assert h.strips()["strips"] and h.strips(transpose=True)["strips"]
            assert bits_equal(h.solve_t(b), ref.solve_t(b)) and bits_equal(h.solve(b), ref.solve(b))
        h.configure(algo=1)
        h.update_values(d[2])
        h.configure(algo=0)
        g = h.capture(b, y, stream=s)                    # captured while the copy is old
        for k in range(3):
            v = d[2] * (2.0 + k)
            h.configure(algo=1)
            h.update_values(v)
            ref.update_values(v)
            g.launch(s)
            s.synchronize()
            assert bits_equal(y, ref.solve(b))
            h.configure(algo=0)
            assert bits_equal(h.solve(b), ref.solve(b))
        h.status()


def test_cooperative_option_costs_strips_nothing(sp):
    """Strips need no co-residency, so the option leaves their launch alone (a
    cooperative one took 125 us instead of 21)."""
    T = W.laplacian_triangle((64, 64))
    d, b = dev_tri(T), dev(W.uniform_vector(T.n, 3))

    def us(**o):
        h = sp.Handle(*d).configure(**o)
        assert h.strips()["strips"]
        best = 1e9
        for _ in range(5):
            t0, t1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            h.solve(b)
            t0.record()
            for _ in range(40):
                h.solve(b)
            t1.record()
            t1.synchronize()
            best = min(best, t0.elapsed_time(t1) / 40 * 1e3)
        h.status()
        return best
    assert us(cooperative=1) < 2 * us()


def test_first_solves_of_shallow_triangles_under_capture(sp):
    """Captured right after the analysis (T^T: after prepare_transpose), without a
    solve before, whatever form they take; replays beside the handle's own solves."""
    chains = band(16384, [1])
    rows = np.repeat(np.arange(16384), np.diff(chains.row_ptr))
    cut = (chains.col_idx % 256 != 255) | (chains.col_idx == rows)
    rp = np.concatenate([[0], np.cumsum(np.add.reduceat(cut, chains.row_ptr[:-1]))]).astype(np.int32)
    for T in (W.laplacian_triangle((3, 3)), band(20000, []), W.laplacian_triangle((40, 30)),
              W.Triangle(16384, rp, chains.col_idx[cut], chains.vals[cut])):
        d, b = dev_tri(T), dev(W.uniform_vector(T.n, 7))
        one = sp.Handle(*d).configure(algo=1, group=1)
        want, want_t = one.solve(b), one.solve_t(b)
        h = sp.Handle(*d, setup="device")
        h.prepare_transpose()
        y, z = torch.empty_like(b), torch.empty_like(b)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            h.solve(b, out=y)
            h.solve_t(b, out=z)
        for _ in range(3):
            y.zero_()
            z.zero_()
            g.replay()
            torch.cuda.synchronize()
            assert bits_equal(y, want) and bits_equal(z, want_t)
            assert bits_equal(h.solve(2 * b), one.solve(2 * b))
        h.status()
