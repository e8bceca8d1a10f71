"""Sorts through a workspace on streams that have no buffer of their own."""
import threading

import numpy as np
import pytest

from oracle import oracle as O
from paper_1506_01446_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

PER_THREAD = 2  # the handle of the calling thread's own stream


def _bind():
    from paper_1506_01446_amd import binding as B
    return B


@pytest.mark.parametrize("n", [4097, 1 << 14, 1 << 15, (1 << 15) + 1, 1 << 17, (1 << 17) + 1])
def test_per_thread_stream(n):
    """Middle sizes there run the network or a sort by rank, long ones
    digits."""
    B = _bind()
    keys = [W.uniform_i32(n + t, n) for t in range(3)]
    got = [None] * 3

    def work(t):
        k = torch.from_numpy(keys[t].copy()).cuda()
        w = k.to(torch.int64) * 3
        v = torch.arange(n, dtype=torch.int32, device="cuda")
        p = k.clone()
        torch.cuda.synchronize()
        B.bitonic_sort_i32(k, True, stream=PER_THREAD)
        B.bitonic_sort_keys64(w, False, stream=PER_THREAD)
        B.bitonic_sort_pairs(p, v, True, stream=PER_THREAD)
        torch.cuda.synchronize()
        got[t] = [x.cpu().numpy() for x in (k, w, p, v)]

    threads = [threading.Thread(target=work, args=(t,)) for t in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for t in range(3):
        k, w, p, v = got[t]
        want = O.sort_i32(keys[t], True)
        assert np.array_equal(k, want)
        assert np.array_equal(w, want[::-1].astype(np.int64) * 3)
        assert np.array_equal(p, want)
        assert np.array_equal(v, np.argsort(keys[t], kind="stable").astype(np.int32))


def test_streams_that_come_and_go():
    """More streams than buffers are kept for, destroyed after use: sorts by
    rank and by digits on each."""
    import ctypes
    B = _bind()
    B.load()
    rt = ctypes.CDLL("libamdhip64.so.7")   # the runtime the process has loaded
    sizes = (6000, 140_001)
    keys = {n: W.uniform_i32(n, n) for n in sizes}
    want = {n: O.sort_i32(keys[n], True) for n in sizes}
    for r in range(3):
        streams = []
        for _ in range(40):
            h = ctypes.c_void_p()
            assert rt.hipStreamCreateWithFlags(ctypes.byref(h), 1) == 0
            streams.append(h)
        work = [(n, torch.from_numpy(keys[n].copy()).cuda()) for n in sizes for _ in streams]
        torch.cuda.synchronize()
        for i, (n, t) in enumerate(work):
            B.bitonic_sort_i32(t, True, stream=streams[i % 40].value)
        torch.cuda.synchronize()
        for n, t in work:
            assert np.array_equal(t.cpu().numpy(), want[n]), (r, n)
        for h in streams:
            assert rt.hipStreamDestroy(h) == 0


def test_workspaces_are_given_back():
    """The memory a large sort leaves with the library comes back."""
    B = _bind()
    n = 50_000_000
    B.bitonic_release_workspaces()
    t = torch.randint(-2**31, 2**31 - 1, (n,), dtype=torch.int32, device="cuda")
    want = t.sort().values
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    B.bitonic_sort_i32(t, True)
    torch.cuda.synchronize()
    assert torch.cuda.mem_get_info()[0] <= before - 4 * n
    B.bitonic_release_workspaces()
    assert torch.cuda.mem_get_info()[0] >= before - (32 << 20)
    assert torch.equal(t, want)
    t = t.flip(0).contiguous()
    B.bitonic_sort_i32(t, True)
    assert torch.equal(t, want)
