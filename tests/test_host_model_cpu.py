"""The library's host side on the CPU, over a stand-in HIP runtime (see
cpp/host_model.cpp): which form a call takes, what it leaves allocated, and what
error it leaves behind, also where allocations fail or a stream is capturing."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1710_04985_amd", "csrc")
MB = 1 << 20
OPT = {"algo": 0, "group": 1, "wg": 7, "assign": 9, "poll": 10, "multi_rows": 12}
P, I32, I64 = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64


@pytest.fixture(scope="module")
def built(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("model") / "host_model.so")
    src = [os.path.join(CSRC, f) for f in ("api.cpp", "devmem.cpp", "analysis.cpp", "strips.cpp")]
    subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-Wl,-Bsymbolic",
                    "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", CSRC,
                    "-I", os.path.join(ROOT, "include"), *src,
                    os.path.join(ROOT, "tests", "cpp", "host_model.cpp"), "-o", out], check=True)
    return out


@pytest.fixture
def m(built, tmp_path):
    """A fresh copy, so that no state of the process-wide kind is shared."""
    path = str(tmp_path / "m.so")
    with open(built, "rb") as a, open(path, "wb") as b:
        b.write(a.read())
    lib = ctypes.CDLL(path)
    for f in (lib.model_fail_from, lib.model_npub, lib.model_strip_bytes):
        f.argtypes = [I64]
    lib.model_alloc.argtypes, lib.model_alloc.restype = [I64], P
    lib.model_xp.restype = P
    lib.model_free.argtypes = lib.model_is_live.argtypes = [P]
    lib.model_live_bytes.restype = I64
    lib.model_log.restype = ctypes.c_char_p
    lib.log = lambda: lib.model_log().decode().split()
    lib.model_fail_from(-1)
    return lib


class Model:
    """A handle over the stand-in runtime."""

    def __init__(self, m, T, nrhs=64):
        self.m, self.n, self.T = m, T.n, T
        self.rp = np.ascontiguousarray(T.row_ptr, np.int32)
        self.ci = np.ascontiguousarray(T.col_idx, np.int32)
        self.v = np.ascontiguousarray(T.vals, np.float64)
        self.b = np.ones(T.n * nrhs)
        self.x = np.zeros(T.n * nrhs)
        self.h = P()
        self.st = m.sptrsv_analyze_ex(I32(T.n), I32(T.nnz), self.p(self.rp), self.p(self.ci),
                                      self.p(self.v), 0, int(T.upper), 0, 0, None,
                                      ctypes.byref(self.h))

    @staticmethod
    def p(a):
        return a.ctypes.data_as(P)

    def set(self, **kw):
        for k, v in kw.items():
            assert self.m.sptrsv_set_option(self.h, OPT[k], I64(v)) == 0
        return self

    def solve(self, t=False):
        f = self.m.sptrsv_solve_transpose if t else self.m.sptrsv_solve
        return f(self.h, self.p(self.b), self.p(self.x), None)

    def multi(self, nrhs, t=False):
        return self.m.sptrsv_solve_multi(self.h, I32(nrhs), I32(self.n), self.p(self.b),
                                         self.p(self.x), int(t), None)

    def update(self):
        """The launches of a value update."""
        self.m.log()
        assert self.m.sptrsv_update_values(self.h, self.p(self.v), None) == 0
        return self.m.log()

    def tune(self, nrhs=1):
        y = np.zeros(self.n * nrhs)
        if nrhs > 1:
            return self.m.sptrsv_tune_multi(self.h, I32(nrhs), I32(self.n), self.p(self.b), self.p(y), None)
        return self.m.sptrsv_tune(self.h, self.p(self.b), self.p(y), None)

    def form(self, nrhs=1, t=False):
        """The launch that a solve comes down to."""
        self.m.log()
        assert (self.multi(nrhs, t) if nrhs > 1 else self.solve(t)) == 0
        return [w for w in self.m.log() if w not in ("fill", "multi_in", "multi_out")][-1]

    def destroy(self):
        assert self.m.sptrsv_destroy(self.h) == 0


def test_allocation_that_succeeds_after_the_store_is_emptied(m):
    a = m.model_alloc(4 * MB)
    m.model_free(a)
    assert m.model_live_bytes() == 4 * MB              # kept
    m.model_fail_next(1)
    b = m.model_alloc(8 * MB)
    assert b and m.model_live_bytes() == 8 * MB        # the kept block went back
    assert m.model_last_error() == 0
    small = m.model_alloc(4 * MB)
    m.model_free(small)
    m.model_fail_next(1)
    assert m.model_alloc(100) and m.model_last_error() == 0


def test_failed_allocations_leave_no_error_behind(m):
    m.model_fail_from(MB)
    assert not m.model_alloc(16 * MB) and m.model_last_error() == 0
    m.model_fail_from(1)
    assert not m.model_alloc(10) and m.model_last_error() == 0
    m.model_fail_from(-1)
    a = m.model_alloc(2 * MB)
    m.model_fail_from(1)                               # no memory for the wait of a free either
    m.model_free(a)
    assert m.model_live_bytes() == 0 and m.model_last_error() == 0


def test_no_memory_for_the_strips(m):
    """Analysis without room for the strip-ordered copy keeps the row-wise
    schedules, and the next launch sees no error; an error of the runtime is
    not taken for that."""
    T = W.laplacian_triangle((128, 128))
    m.model_strip_bytes(64 * MB)
    m.model_fail_from(32 * MB)
    h = Model(m, T)
    assert h.st == 0 and m.model_last_error() == 0
    m.log()
    assert h.solve() == 0 and m.log()[-1] != "strips"
    assert h.solve(t=True) == 0 and m.log()[-1] != "strips"
    h.destroy()
    m.model_fail_from(-1)
    h = Model(m, T)
    assert h.st == 0 and h.solve() == 0 and m.log()[-1] == "strips"
    h.destroy()
    m.model_strip_error(-8)
    assert Model(m, T).st == -8


def test_no_memory_for_the_strips_buffer(m):
    """Several columns whose published values do not fit in memory, where those
    of the row-wise solve do, are solved row-wise; with memory, in strips.  A
    default block choice builds its plan then."""
    T = W.laplacian_triangle((128, 128))
    m.model_npub(16 * T.n)
    h = Model(m, T)
    m.log()
    m.model_fail_from(16 * MB)
    assert h.multi(16) == 0 and m.log()[-1] == "multi_out"
    assert h.multi(16, t=True) == 0 and m.log()[-1] == "multi_out"
    assert m.model_last_error() == 0
    m.model_fail_from(-1)
    assert h.multi(16) == 0 and m.log()[-1] == "strips"
    h.destroy()

    T = W.laplacian_triangle((40, 40))
    h = Model(m, T)                                    # room for T's values only
    m.model_npub(64 << 20)
    m.model_fail_from(16 * MB)
    assert h.solve(t=True) == 0 and m.log()[-1] == "block"


@pytest.mark.parametrize("later", ["transpose", "columns"])
def test_buffer_in_a_capture_of_the_callers_own(m, later):
    """A buffer whose address a caller's graph holds outlives the call that
    needs a larger one, and goes with the handle."""
    T = W.laplacian_triangle((50, 50))
    h = Model(m, T).set(algo=2)
    assert h.solve() == 0
    m.model_capture(1)
    assert h.solve() == 0
    m.model_capture(0)
    held = m.model_xp()
    m.model_npub(4 * T.n)                              # T^T publishes more
    assert (h.solve(t=True) if later == "transpose" else h.multi(4)) == 0
    assert m.model_xp() != held and m.model_is_live(held)
    h.destroy()
    assert not m.model_is_live(held) and m.model_live_bytes() == 0


@pytest.mark.parametrize("order", [(64, 256), (256, 64)])
def test_tuned_choice_of_another_workgroup_size(m, order):
    """A choice kept for a pattern is one of a handle with the same candidates."""
    T = W.laplacian_triangle((60, 50))
    for wg in order:
        h = Model(m, T).set(algo=2, wg=wg)
        assert h.tune() == 0
        assert (h.form() == "strips") == (wg == 64)
        if wg == 64:
            assert h.set(wg=128).form() != "strips"     # set after the tuning


def test_tuned_columns_respect_the_rows_option(m):
    T = W.laplacian_triangle((60, 50))
    h = Model(m, T).set(algo=2, multi_rows=2)
    assert h.tune(4) == 0 and h.form(4) != "strips"
    h.set(multi_rows=0)
    assert h.tune(4) == 0 and h.form(4) == "strips"
    assert h.set(wg=128).form(4) != "strips"


def _rows(n, pairs):
    """Unit-pattern triangle with the given (rows, columns) off the diagonal."""
    i = np.arange(n, dtype=np.int64)
    key = np.unique(np.concatenate([i * n + i] + [r * n + c for r, c in pairs]))
    rp = np.zeros(n + 1, np.int64)
    np.cumsum(np.bincount(key // n, minlength=n), out=rp[1:])
    return W.Triangle(n, rp.astype(np.int32), (key % n).astype(np.int32), np.ones(key.size))


def _chains(n, length):
    i = np.arange(n, dtype=np.int64)
    k = i[i % length != 0]
    return _rows(n, [(k, k - 1)])


def _offset(n, *offsets):
    return _rows(n, [(np.arange(o, n, dtype=np.int64), np.arange(n - o, dtype=np.int64)) for o in offsets])


def _half(n):
    i = np.arange(n // 2, n, dtype=np.int64)
    return _rows(n, [(i, i - n // 2), (i[1:], i[1:] - n // 2 - 1)])


def _planes(side):
    """Layers of a 3-D grid that do not depend on one another: reads as a 2-D
    grid of side x side^2."""
    i = np.arange(side ** 3, dtype=np.int64)
    x, y = i % side, i // side % side
    return _rows(side ** 3, [(i[x > 0], i[x > 0] - 1), (i[y > 0], i[y > 0] - side)])


# wide, shallow triangles on grid-like offsets: far fewer levels than a line has rows
SHALLOW = {"independent": _rows(20000, []), "independent_few": _rows(500, []),
           "far_offset": _offset(400000, 100000), "chains": _chains(16384, 256),
           "short_chains": _chains(20000, 10), "two_colours": _half(60000), "planes": _planes(64)}


@pytest.mark.parametrize("name", SHALLOW)
def test_shallow_triangles_are_solved_row_wise(m, name):
    h = Model(m, SHALLOW[name])
    for t in (False, True):
        for nrhs in (1, 8):
            assert h.form(nrhs, t) != "strips", (t, nrhs)
    h.set(algo=2)
    assert h.form() != "strips"


def test_deep_triangles_are_solved_in_strips(m):
    """Also where only some directions of the grid, or some entries, are there."""
    rng = np.random.Generator(np.random.PCG64(1))
    T = W.laplacian_triangle((96, 96))
    rows = np.repeat(np.arange(T.n, dtype=np.int64), np.diff(T.row_ptr))
    k = rng.random(T.nnz) < 0.5
    for T in (W.laplacian_triangle((64, 64)), W.laplacian_triangle((20, 30, 16)), _offset(100000, 1000),
              _offset(300000, 5000), _chains(3000, 3000), _chains(3000, 500),
              _rows(T.n, [(rows[k], T.col_idx[k].astype(np.int64))])):
        h = Model(m, T)
        assert h.form() == "strips" and h.form(8) == "strips" and h.form(t=True) == "strips"


def test_tiny_triangles_take_one_launch(m):
    for T in (_chains(5, 5), W.laplacian_triangle((4, 4)), W.laplacian_triangle((1, 1))):
        assert Model(m, T).form() == "block"
    assert Model(m, W.laplacian_triangle((16, 16))).form() == "strips"


def test_batches_of_many_small_systems(m):
    """Strips cost a claim each, so many small systems keep the row-wise form,
    more so with several columns."""
    def batch(side, count):
        return W.concat_block_diagonal([W.laplacian_triangle((side, side))] * count)

    def form(side, count, nrhs, offsets=True):
        T = batch(side, count)
        m.log()
        n1, z1 = side * side, T.nnz // count
        one = W.laplacian_triangle((side, side))
        rp, ci, v = (np.ascontiguousarray(a, t) for a, t in
                     ((one.row_ptr, np.int32), (one.col_idx, np.int32), (one.vals, np.float64)))
        h = Model.__new__(Model)
        h.m, h.n, h.h = m, T.n, P()
        h.b, h.x = np.ones(T.n * 16), np.zeros(T.n * 16)
        arr = lambda a: (P * count)(*[a.ctypes.data] * count)
        assert m.sptrsv_analyze_batched_ex(I32(count), (I32 * count)(*[n1] * count),
                                           (I32 * count)(*[z1] * count), arr(rp), arr(ci), arr(v), 0,
                                           0, 0, 0, None, ctypes.byref(h.h)) == 0
        assert ("offsets" in m.log()) == offsets
        out = h.form(nrhs)
        h.destroy()
        return out
    assert form(8, 4000, 1) != "strips"
    # so many, so small: whatever they look like
    assert form(2, 4000, 1, offsets=False) != "strips" and form(3, 1500, 1, offsets=False) != "strips"
    assert form(16, 300, 16) != "strips"
    assert form(32, 64, 1) == "strips" and form(32, 64, 8) == "strips"


def _layers(n, layers, near, far):
    """Rows with `near` entries in the layer above and `far` in those three and
    more up, at random."""
    w = n // layers
    rng = np.random.Generator(np.random.PCG64(2))
    i = np.arange(w, n, dtype=np.int64)
    pairs = [(i, (i // w - 1) * w + rng.integers(0, w, i.size)) for _ in range(near)]
    k = i[i >= 4 * w]
    pairs += [(k, (k // w - 3) * w - 1 - rng.integers(0, w, k.size)) for _ in range(far)]
    return _rows(n, pairs)


def test_rows_published_one_by_one_where_they_wait_for_little(m):
    """The static row-wise schedule publishes by row where few entries of a lane
    are one level up, and by chunk where most are."""
    for T, want in ((_layers(20000, 20, 8, 0), "static"), (_layers(20000, 20, 16, 0), "static"),
                    (_layers(20000, 20, 1, 7), "static_by_row"), (_layers(30000, 20, 2, 14), "static"),
                    (_layers(100000, 11, 4, 4), "static_by_row"),     # wide layers
                    (_layers(40000, 20, 4, 4), "static"), (_layers(40000, 20, 1, 39), "static_by_row"),
                    (W.powerlaw_lower(20000, 3, window=2000), "static_by_row"),
                    (W.stencil_triangle((20, 20, 20), 27), "static"),
                    (W.laplacian_triangle((30, 30, 30)), "static")):
        h = Model(m, T).set(algo=2, assign=0)
        assert h.form() == want
        assert h.set(poll=0).form() == "static"


def test_value_updates_follow_the_form_that_is_used(m):
    """New values go to the strip-ordered copies where solves read them: at
    once, or with the first solve that needs them; a captured solve or update
    always finds them current."""
    T = W.laplacian_triangle((64, 64))
    h = Model(m, T)
    assert h.solve(t=True) == 0
    assert h.update()[-2:] == ["strip_gather", "strip_gather"]
    h.set(algo=1)
    assert "strip_gather" not in h.update()
    h.set(algo=0)
    m.log()
    assert h.solve() == 0 and m.log() == ["strip_gather", "fill", "strips"]
    assert h.solve() == 0 and m.log() == ["fill", "strips"]
    assert h.solve(t=True) == 0 and m.log() == ["strip_gather", "fill", "strips"]
    h.set(algo=1)
    assert "strip_gather" not in h.update()
    m.model_capture(1)
    assert h.update().count("strip_gather") == 2       # the graph's
    m.model_capture(0)
    h.set(algo=0)
    m.log()
    assert h.solve() == 0 and m.log()[0] == "strip_gather"      # the graph has not run
    h.set(algo=1)
    assert "strip_gather" not in h.update()
    h.set(algo=0)
    m.log()
    m.model_capture(1)
    assert h.solve() == 0 and m.log()[0] == "strip_gather"
    m.model_capture(0)
    h.set(algo=1)
    assert h.update().count("strip_gather") == 1       # that graph's copy stays current
    h.set(algo=0)
    m.log()
    assert h.solve() == 0 and m.log() == ["fill", "strips"]


def test_kept_memory_is_given_back_on_request(m):
    h = Model(m, W.laplacian_triangle((300, 300)))
    assert h.st == 0
    h.destroy()
    assert m.model_live_bytes() > 0
    assert m.sptrsv_release_memory() == 0 and m.model_live_bytes() == 0
    assert m.sptrsv_release_memory() == 0
    a = m.model_alloc(3 * MB)                          # what is in use stays
    m.model_free(m.model_alloc(5 * MB))
    assert m.sptrsv_release_memory() == 0 and m.model_live_bytes() == 4 * MB and m.model_is_live(a)


def test_blocks_that_a_reset_took_are_not_handed_out(m):
    for _ in range(3):
        m.model_free(m.model_alloc(6 * MB))
    m.model_reset()
    a = m.model_alloc(6 * MB)
    assert a and m.model_is_live(a) and m.model_last_error() == 0


def test_allocations_of_a_capture_keep_the_store(m):
    """A refused allocation under capture is no lack of memory: nothing is taken
    out of the store that could not be freed."""
    m.model_free(m.model_alloc(4 * MB))
    m.model_capture(1)
    assert not m.model_alloc(64 * MB)
    m.model_capture(0)
    assert m.sptrsv_release_memory() == 0 and m.model_live_bytes() == 0


@pytest.mark.parametrize("by", ["bound", "want", "request"])
def test_other_threads_allocate_while_blocks_go_back(m, by):
    """Freeing a block waits for its device; another thread's allocation does
    not wait with it."""
    blocks = [m.model_alloc(700 * MB), m.model_alloc(600 * MB)]
    m.model_free(blocks[0])
    m.model_probe_free()
    if by == "bound":
        m.model_free(blocks[1])
    elif by == "want":
        m.model_fail_next(1)
        assert m.model_alloc(900 * MB)
    else:
        assert m.sptrsv_release_memory() == 0
    assert m.model_probed() == 2


def test_small_host_patterns_are_read_on_the_host(m):
    for T, want in ((W.laplacian_triangle((60, 60)), True), (W.powerlaw_lower(2000, 3, window=300), False),
                    (W.laplacian_triangle((200, 200)), None)):
        m.log()
        h = Model(m, T)
        assert h.st == 0 and ("offsets" in m.log()) == (want is None)
        assert (h.form() == "strips") == (want is not False)


def test_first_solves_under_capture(m):
    """A captured solve needs no table that is not there yet: T after the
    analysis, T^T after sptrsv_prepare_transpose, also where T^T is not solved in
    strips; and several columns in strips where the row-wise tables are missing."""
    for T in (_chains(5, 5), W.laplacian_triangle((4, 4)), W.laplacian_triangle((60, 60)), SHALLOW["chains"],
              SHALLOW["independent"], W.laplacian_triangle((20, 20, 20))):
        h = Model(m, T)
        assert m.sptrsv_prepare_transpose(h.h, None) == 0
        m.model_capture(1)
        assert h.solve() == 0 and h.solve(t=True) == 0, T.n
        m.model_capture(0)
        h.destroy()
    # strips win for one column and lose for sixteen: captured, they are there
    rng = np.random.Generator(np.random.PCG64(1))
    T = W.laplacian_triangle((128, 128))
    rows = np.repeat(np.arange(T.n, dtype=np.int64), np.diff(T.row_ptr))
    k = rng.random(T.nnz) < 0.2
    h = Model(m, _rows(T.n, [(rows[k], T.col_idx[k].astype(np.int64))]))
    m.model_npub(100)
    assert m.sptrsv_prepare_transpose(h.h, None) == 0
    assert h.form() != "strips" and h.form(16) == "strips"
