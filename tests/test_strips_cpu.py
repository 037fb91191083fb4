"""The strip form's grids, strips and LDS ring on the CPU: every row on one
line, every entry at the ring place the kernel would read it from, for ghost
values brought in as late and as early as the kernel may."""
import ctypes
import os
import subprocess
import time

import numpy as np
import pytest

import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1710_04985_amd", "csrc")


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    out = tmp_path_factory.mktemp("strips") / "strip_check.so"
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-I", CSRC,
                    os.path.join(ROOT, "tests", "cpp", "strip_check.cpp"),
                    os.path.join(CSRC, "strips.cpp"), "-o", str(out)], check=True)
    lib = ctypes.CDLL(str(out))

    def run(T, attempt=0, cut=0, fn=lib.check_strips):
        n = T.n - cut                                   # a leading (lower) part: a cut last line
        rp = np.ascontiguousarray(T.row_ptr[:n + 1], np.int32)
        ci = np.ascontiguousarray(T.col_idx[:rp[-1]], np.int32)
        p = lambda a: a.ctypes.data_as(ctypes.c_void_p)
        return fn(n, p(rp), p(ci), int(T.upper), attempt)
    run.lib = lib
    run.levels = lambda T, **o: run(T, fn=lib.check_levels, **o)
    return run


GRIDS = [((1, 1), 5), ((2, 3), 5), ((64, 64), 5), ((65, 63), 5), ((63, 130), 9), ((200, 7), 9),
         ((5, 300), 9), ((9, 7, 5), 7), ((33, 20, 17), 7), ((70, 3, 40), 7), ((2, 2, 50), 7),
         ((16, 16, 200), 7), ((12, 11, 13), 27), ((4, 33, 6), 27), ((40, 5, 9), 27), ((9, 8, 120), 27)]


@pytest.mark.parametrize("upper", [False, True])
@pytest.mark.parametrize("dims,points", GRIDS, ids=["x".join(map(str, g)) + "_%d" % p for g, p in GRIDS])
def test_grids(check, dims, points, upper):
    T = W.stencil_triangle(dims, points, upper=upper)
    assert check(T) == 0
    assert check.levels(T) == 0
    if not upper and T.n > 10:
        assert check(T, cut=3) == 0


def test_patterns_that_are_no_grid(check):
    # more offsets than a stencil; offsets no strides explain; entries that
    # run across the line ends of the grid their offsets suggest
    assert check(W.powerlaw_lower(3000, 1, window=500)) == -1
    i = np.arange(900)

    def band(offsets):
        cols = [[r - o for o in sorted(offsets, reverse=True) if r >= o] + [r] for r in i]
        rp = np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int32)
        return W.Triangle(900, rp, np.concatenate(cols).astype(np.int32), np.ones(rp[-1]))
    assert check(band([2, 5, 7])) != 0
    assert check(band([1, 30])) == 4
    assert check(band([29, 30]), attempt=1) in (0, 4)


def test_second_reading_of_a_cluster_of_two_offsets(check):
    """Offsets 29 and 30: a grid of 29 columns whose entries reach back over
    line ends on the first reading, one of 30 on the second; neither fits."""
    i = np.arange(900)
    cols = [[r - o for o in (30, 29) if r >= o] + [r] for r in i]
    rp = np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int32)
    T = W.Triangle(900, rp, np.concatenate(cols).astype(np.int32), np.ones(rp[-1]))
    assert check(T) == 4 and check(T, attempt=1) == 4


def band(n, offsets):
    """Rows with an entry at each offset (each divides the next) unless it would
    lie beyond the start of the row's line or plane."""
    i = np.arange(n)
    ends = list(offsets[1:]) + [n]
    has = [i % e >= o for o, e in zip(offsets, ends)]
    r = np.concatenate([i] + [i[k] for k in has])
    c = np.concatenate([i] + [i[k] - o for k, o in zip(has, offsets)])
    order = np.lexsort((c, r))
    rp = np.zeros(n + 1, np.int64)
    np.cumsum(np.bincount(r, minlength=n), out=rp[1:])
    return W.Triangle(n, rp.astype(np.int32), c[order].astype(np.int32), np.ones(r.size))


@pytest.mark.parametrize("n,offsets", [(7000, [1000]), (7321, [1000]), (30000, [5000]), (4096, [64, 1024]),
                                       (4001, [64, 1024]), (6000, [1, 600]), (9000, [100])])
def test_lines_without_coupling(check, n, offsets):
    """Entries one line or plane back only: the walk follows them, the lines
    that do not depend on one another lie across the lanes."""
    T = band(n, offsets)
    assert check(T) == 0
    assert check.levels(T) == 0
    assert check(_transposed(T)) == 0


def _transposed(T):
    rows = np.repeat(np.arange(T.n), np.diff(T.row_ptr))
    order = np.lexsort((rows, T.col_idx))
    rp = np.zeros(T.n + 1, np.int64)
    np.cumsum(np.bincount(T.col_idx, minlength=T.n), out=rp[1:])
    return W.Triangle(T.n, rp.astype(np.int32), rows[order].astype(np.int32), T.vals[order], upper=True)


STENCILS = {"5": [(0, 1, 0), (1, 0, 0)], "9": [(0, 1, 0)] + [(1, a, 0) for a in (-1, 0, 1)],
            "7": [(0, 1, 0), (1, 0, 0), (0, 0, 1)],
            "27": [(0, 1, 0)] + [(1, a, 0) for a in (-1, 0, 1)] +
                  [(b, a, 1) for b in (-1, 0, 1) for a in (-1, 0, 1)]}


@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("upper", [False, True])
@pytest.mark.parametrize("dims,stencil", [((9, 6, 1), "5"), ((7, 8, 1), "9"), ((5, 6, 4), "7"), ((5, 4, 6), "27")])
def test_runs_of_cut_lines(check, dims, stencil, upper, axis):
    """The rows on a line, in closed form, where n cuts the last line or plane
    anywhere."""
    sy, sz = dims[0], dims[0] * dims[1]
    offs = np.array(sorted(b * sy + a + c * sz for b, a, c in STENCILS[stencil]), np.int32)
    for n in range(sz * (dims[2] - 1) + 1 if dims[2] > 1 else 2 * sy + 1, sz * dims[2] + 1):
        rc = check.lib.check_lines(n, offs.ctypes.data_as(ctypes.c_void_p), offs.size, int(upper), axis, 0)
        assert rc == 0, n


@pytest.mark.parametrize("upper", [False, True])
def test_long_cut_lines_take_no_search(check, upper):
    offs = np.array([1, 500000000], np.int32)
    t0 = time.perf_counter()
    for _ in range(100):
        assert check.lib.check_lines(500000010, offs.ctypes.data_as(ctypes.c_void_p), 2, int(upper), 0, 2) == 0
    assert time.perf_counter() - t0 < 1.0              # a search takes seconds for one
