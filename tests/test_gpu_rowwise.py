"""The static row-wise schedule where rows of several lanes exist (each row is
published as soon as its own dependencies have come): row lengths at the edges
of the lane groups, in one triangle, against the level-scheduled solve bit for
bit and against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import workloads as W
from gpuhelp import bits_equal, dev, dev_tri, host, relerr

pytestmark = pytest.mark.gpu

LENGTHS = [0, 1, 3, 4, 5, 8, 9, 16, 17, 32, 33, 64, 65, 128, 129, 255, 256, 257, 300]


@pytest.fixture(scope="module")
def sp():
    import paper_1710_04985_amd as sp
    assert torch.cuda.is_available()
    return sp


def _rows(n, lengths, window, seed, upper=False):
    """Rows of the given lengths in turn, columns drawn from the window below."""
    rng = np.random.Generator(np.random.PCG64(seed))
    rp, cols, vals = [0], [], []
    for i in range(n):
        lo = max(0, i - window)
        k = min(lengths[rng.integers(len(lengths))], i - lo)
        c = np.sort(lo + rng.choice(i - lo, k, replace=False)) if k else np.zeros(0, int)
        cols += list(c) + [i]
        vals += list(rng.uniform(-1, 1, k) / max(k, 1)) + [rng.uniform(1, 2)]
        rp.append(len(cols))
    rp, cols, vals = np.array(rp), np.array(cols), np.array(vals)
    if upper:                                             # the same, backwards
        rows = np.repeat(np.arange(n), np.diff(rp))
        rp = np.concatenate([[0], np.cumsum(np.diff(rp)[::-1])])
        cols, vals = n - 1 - cols[::-1], vals[::-1]
    return W.Triangle(n, rp.astype(np.int32), cols.astype(np.int32), vals, upper=upper)


CASES = [(3000, LENGTHS, 400, False), (2500, LENGTHS, 2500, True), (4000, [0, 1, 4, 5], 70, False),
         (700, [64, 256], 700, False), (1, [0], 5, False), (66, [5], 5, True)]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("n,lengths,window,upper", CASES, ids=["%d_%d" % (c[0], c[2]) for c in CASES])
def test_rows_published_one_by_one(sp, n, lengths, window, upper, dtype):
    T = _rows(n, lengths, window, 11, upper)
    b = dev(W.uniform_vector(n, 4), dtype)
    uplo = "U" if upper else "L"
    d = dev_tri(T, dtype)
    ref = sp.Handle(*d, uplo=uplo).configure(algo=1)
    want, want_t = ref.solve(b), ref.solve_t(b)
    for o in ({}, {"grid": 1}, {"grid": 3, "assign": 0}, {"xp_stride": 8}, {"poll": 0}, {"wg": 256}):
        h = sp.Handle(*d, uplo=uplo).configure(algo=2, **{"assign": 2, **o})
        for _ in range(3):
            assert bits_equal(h.solve(b), want) and bits_equal(h.solve_t(b), want_t)
        h.status()
    x = oracle.get().solve(T.row_ptr, T.col_idx, host(d[2]).astype(np.float64),
                           host(b).astype(np.float64), upper)
    assert relerr(host(want), x) <= (1e-12 if dtype == torch.float64 else 1e-5)


def test_special_values_reach_their_rows_only(sp):
    """Infinities, NaN and signed zeros in b: absent entries change nothing."""
    T = _rows(2000, [0, 1, 2, 4, 5, 7, 9], 60, 12)
    b = W.uniform_vector(T.n, 5)
    b[[3, 700]], b[[40, 900]], b[500], b[100:140] = np.inf, -np.inf, np.nan, -0.0
    b = dev(b)
    want = sp.Handle(*dev_tri(T)).configure(algo=1).solve(b)
    h = sp.Handle(*dev_tri(T)).configure(algo=2, assign=2)
    for _ in range(3):
        assert bits_equal(h.solve(b), want)
    h.status()
