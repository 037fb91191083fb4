"""Device memory that outlives a handle: bounded, and safe to reuse from several
threads and streams."""
import threading

import pytest
import torch

import workloads as W
from gpuhelp import bits_equal, dev, dev_tri

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sp():
    import paper_1710_04985_amd as sp
    assert torch.cuda.is_available()
    return sp


def test_kept_memory_is_bounded(sp):
    """Handles of many sizes, several alive at once: what stays allocated after
    the last one is gone is at most the store's 1 GiB (and small change)."""
    torch.cuda.synchronize()
    free0, own0 = torch.cuda.mem_get_info()[0], torch.cuda.memory_reserved()
    tris = [dev_tri(W.laplacian_triangle((s, s, s))) for s in (20, 30, 45, 60, 80)]
    b = [torch.ones(t[0].numel() - 1, dtype=torch.float64, device="cuda") for t in tris]
    live = []
    for k in range(120):
        i = (k * 7) % len(tris)
        h = sp.Handle(*tris[i], setup=("host", "device")[k % 2])
        h.solve(b[i])
        live.append(h)
        if len(live) > 1 + k % 17:
            live = live[len(live) // 2:]
    del live, h
    torch.cuda.synchronize()
    held = free0 - torch.cuda.mem_get_info()[0] - (torch.cuda.memory_reserved() - own0)
    assert held <= (1 << 30) + (256 << 20)


def test_reuse_from_threads_and_streams(sp):
    tris = [W.laplacian_triangle((s, 64, 64)) for s in (24, 40, 33, 28)]
    devs = [dev_tri(t) for t in tris]
    bs = [dev(W.uniform_vector(t.n, 3)) for t in tris]
    want = [sp.Handle(*d).solve(b) for d, b in zip(devs, bs)]
    torch.cuda.synchronize()
    wrong = []

    def work(k):
        with torch.cuda.stream(torch.cuda.Stream()):
            for r in range(8):
                i = (k + r) % len(tris)
                h = sp.Handle(*devs[i], setup=("device", "host")[r % 4 == 3])
                x = h.solve(bs[i])
                del h                                    # its work may still be running
                if not bits_equal(x, want[i]):
                    wrong.append((k, r))
    ts = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    [t.start() for t in ts]
    [t.join() for t in ts]
    assert not wrong


def test_handle_destroyed_beside_a_relaxed_capture(sp):
    """Giving memory back leaves another stream's capture alone where the
    capture allows calls like hipFree."""
    T = W.laplacian_triangle((48, 48, 48))
    d, b = dev_tri(T), dev(W.uniform_vector(T.n, 3))
    h = sp.Handle(*d)
    want = h.solve(b)
    a = torch.arange(1000.0, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, capture_error_mode="relaxed"):
        c = a * 2
        del h
        e = c + 1
    for _ in range(3):
        e.zero_()
        g.replay()
        assert torch.equal(e, a * 2 + 1)
    assert bits_equal(sp.Handle(*d).solve(b), want)


def test_kept_memory_is_given_back_on_request(sp):
    d = dev_tri(W.laplacian_triangle((90, 90, 90)))
    b = torch.ones(d[0].numel() - 1, dtype=torch.float64, device="cuda")
    sp.release_memory()
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    h = sp.Handle(*d, setup="device")
    x = h.solve(b)
    del h
    torch.cuda.synchronize()
    kept = free0 - torch.cuda.mem_get_info()[0]
    sp.release_memory()
    assert kept > (50 << 20) and free0 - torch.cuda.mem_get_info()[0] < (32 << 20)
    assert bits_equal(sp.Handle(*d, setup="device").solve(b), x)
