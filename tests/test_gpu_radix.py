"""The digit sorts of long single arrays against the CPU oracle, bit for
bit: every storage and key type, both directions, the sizes where the route,
the tile, its groups and supergroups change, passes that are left out, and
the calls that must keep to the network."""
import threading

import numpy as np
import pytest

from oracle import oracle as O
from paper_1506_01446_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# Sizes: one above the route's start; the tiles' changes (4-byte 2^20 and
# 2^22, 8-byte 2^19 and 2^20); a whole last tile, one element over and one
# short; group (16 tiles) and supergroup (256 tiles) edges of the tile in use.
SIZES32 = [(1 << 15) + 1, (1 << 16) + 1, 16 * 4096, 16 * 4096 + 1, (1 << 20) - 1, 1 << 20,
           (1 << 20) + 1, 1 << 22, (1 << 22) + 1, (1 << 22) + 16 * 16384 - 1]
SIZES64 = [(1 << 15) + 1, 16 * 2048 + 2048, (1 << 19) - 1, 1 << 19, (1 << 20) - 1, (1 << 20) + 1,
           (1 << 21) + 1]


def _bind():
    from paper_1506_01446_amd import binding as B
    return B


def _gpu(a):
    return torch.from_numpy(a.copy()).cuda()


def _words(kind, n, seed):
    """n 64-bit words with the digits a pass can meet: all of them, few
    values, one value, order, and digits that never change."""
    w = W.splitmix64(seed, 0, n).view(np.int64)
    if kind == "few":
        return w[(W.splitmix64(seed + 1, 0, n) >> np.uint64(61)).astype(np.int64)]
    if kind == "equal":
        return np.full(n, w[0])
    if kind == "sorted":
        return np.sort(w)
    if kind == "narrow":     # two digits of either half vary
        return w & np.int64(0x00FF00FF00FF00FF)
    if kind == "one_digit":  # a single digit varies: an odd number of passes
        return w & np.int64(0x0000FF000000FF00)
    return w


KINDS = ["uniform", "few", "equal", "sorted", "narrow", "one_digit"]


@pytest.mark.parametrize("n", SIZES32)
def test_keys32(n):
    B = _bind()
    for i, type_ in enumerate(["int32", "uint32", "float32"]):
        for asc in (True, False):
            k = _words(KINDS[(i + asc + n) % 6], n, n + i).astype(np.int32)
            if type_ == "float32":   # NaNs of both signs, infinities, zeros
                k[:8] = np.array([0x7FC00001, -0x3FFFFF, 0x7F800000, -0x800000, 0, -0x80000000,
                                  1, 0x7FFFFFFF], dtype=np.int64).astype(np.int32)
            t = _gpu(k)
            B.bitonic_sort_keys(t, asc, type_)
            want = O.sort_keys(k.view(type_), i, asc).view(np.int32)
            assert np.array_equal(t.cpu().numpy(), want), (type_, asc)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("offset", [0, 1])
def test_keys32_kinds_and_alignment(kind, offset):
    B = _bind()
    n = 300_001
    k = _words(kind, n + offset, 5).astype(np.int32)
    t = _gpu(k)
    B.bitonic_sort_i32(t[offset:], False)
    got = t.cpu().numpy()
    assert np.array_equal(got[offset:], O.sort_i32(k[offset:], False))
    assert np.array_equal(got[:offset], k[:offset])


@pytest.mark.parametrize("n", SIZES64)
def test_keys64(n):
    B = _bind()
    for i, type_ in enumerate(["int64", "uint64", "float64"]):
        asc = (i + n) % 2 == 0
        k = _words(KINDS[(i + n) % 6], n, n + i).copy()
        if type_ == "float64":
            k[:6] = np.array([0x7FF8000000000001, -1, 0x7FF0000000000000, -(1 << 52), 0,
                              -(1 << 63)], dtype=np.int64)
        t = _gpu(k)
        B.bitonic_sort_keys64(t, asc, type_)
        want = O.sort_keys64(k.view(type_), 3 + i, asc).view(np.int64)
        assert np.array_equal(t.cpu().numpy(), want), (type_, asc)


@pytest.mark.parametrize("n", SIZES64)
@pytest.mark.parametrize("values", ["index", "uniform", "one_step_down", "equal"])
def test_pairs(n, values):
    """Values in order leave the value passes out; one step down anywhere
    (here over the boundary of two counting workgroups) does not."""
    B = _bind()
    for i, type_ in enumerate(["int32", "uint32", "float32"]):
        asc = (i + n) % 2 == 0
        k = _words(["few", "uniform", "one_digit"][(i + n) % 3], n, n + i).astype(np.int32)
        v = np.arange(n, dtype=np.int32) - n // 2
        if values == "uniform":
            v = W.uniform_i32(n + 9, n)
        elif values == "one_step_down":
            v[n // 2:] -= 1
            v[-1] = v[-2] - 1
        elif values == "equal":
            v[:] = -7
        kt, vt = _gpu(k), _gpu(v)
        B.bitonic_sort_pairs(kt, vt, asc, type_)
        wk, wv = O.sort_pairs(k.view(type_), v, i, asc)
        assert np.array_equal(kt.cpu().numpy(), wk.view(np.int32)), (type_, asc)
        assert np.array_equal(vt.cpu().numpy(), wv), (type_, asc)


def test_captured_stream_runs_the_network():
    """A capture takes no workspace: the sort goes into the graph as the
    network, and every replay sorts new keys, with eager sorts between."""
    B = _bind()
    n = (1 << 17) + 5
    buf = torch.empty(n, dtype=torch.int32, device="cuda")
    eager = torch.empty_like(buf)
    B.bitonic_sort_i32(buf, True)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        B.bitonic_sort_i32(buf, True)
    for r in range(3):
        k = W.uniform_i32(50 + r, n)
        buf.copy_(torch.from_numpy(k))
        eager.copy_(torch.from_numpy(k))
        g.replay()
        B.bitonic_sort_i32(eager, True)
        torch.cuda.synchronize()
        want = O.sort_i32(k, True)
        assert np.array_equal(buf.cpu().numpy(), want), r
        assert np.array_equal(eager.cpu().numpy(), want), r


def test_threads_and_streams():
    """Threads that sort on streams of their own and on one they share, sizes
    changing from call to call: each result is the array's own."""
    B = _bind()
    shared = torch.cuda.Stream()
    sizes = [70_001, 1 << 20, 200_000, 3_000_001]
    keys = [[W.uniform_i32(900 + 10 * t + i, n) for i, n in enumerate(sizes)] for t in range(4)]
    got = [[None] * len(sizes) for _ in range(4)]

    def work(t):
        own = torch.cuda.Stream()
        for i in range(len(sizes)):
            st = shared if (t + i) % 2 else own
            with torch.cuda.stream(st):
                d = torch.from_numpy(keys[t][i]).cuda()
                B.bitonic_sort_i32(d, True)
                got[t][i] = d
        own.synchronize()

    threads = [threading.Thread(target=work, args=(t,)) for t in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for t in range(4):
        for i in range(len(sizes)):
            assert np.array_equal(got[t][i].cpu().numpy(), O.sort_i32(keys[t][i], True)), (t, i)
