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
