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

# Sizes: one above the route's start (2^17 keys, 2^16 pairs); the tiles'
# changes (4-byte 2^20 and 2^22, 8-byte 2^19 and 2^20); a whole last tile, one
# element over and one short; group (16 tiles) and supergroup (256 tiles) edges
# of the tile in use.
SIZES32 = [(1 << 17) + 1, 48 * 4096, 48 * 4096 + 1, (1 << 20) - 1, 1 << 20,
           (1 << 20) + 1, 1 << 22, (1 << 22) + 1, (1 << 22) + 16 * 16384 - 1]
SIZES64 = [(1 << 16) + 1, (1 << 17) + 1, 80 * 2048, (1 << 19) - 1, 1 << 19, (1 << 20) - 1,
           (1 << 20) + 1, (1 << 21) + 1]


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
    sizes = [70_001, 1 << 20, 200_000, 3_000_001]  # the first by rank
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


# Segmented sorts: the big segments go by digits when the longest has more
# than 2^17 elements.  Lengths around the small segments' limit (2^13), the
# tiles (2^14, 2^13), a group (16 tiles) and a supergroup (256 tiles: 2^21
# 8-byte elements), with empty segments between.
SEG_LENS = [
    [(1 << 17) + 1, 0, 8193, 5, 8192, 1 << 14, (1 << 14) + 1, 70_001],
    [1 << 18, 1, (1 << 18) + 1, 3 * 8192, 300, 0, 150_000],
    [(1 << 21) + 8193, 20_000, 1 << 17],
]


def _segments(lens, lead):
    off = np.zeros(len(lens) + 1, dtype=np.int64)
    np.cumsum(lens, out=off[1:])
    return off + lead


def _oracle_segments(sort, k, off):
    out = k.copy()
    for a, b in zip(off[:-1], off[1:]):
        out[a:b] = sort(k[a:b])
    return out


@pytest.mark.parametrize("lens", SEG_LENS, ids=["classes", "tiles", "supergroup"])
@pytest.mark.parametrize("bounded", [True, False])
def test_segments(lens, bounded):
    B = _bind()
    off = _segments(lens, 3)      # segments start off a 16-byte boundary
    n = int(off[-1]) + 5
    ot = torch.from_numpy(off).cuda()
    for i, type_ in enumerate(["int32", "uint32", "float32", "int64", "uint64", "float64"]):
        asc = i % 2 == 0
        w = _words(KINDS[(i + len(lens)) % 6], n, 70 + i)
        k = w.copy() if i >= 3 else w.astype(np.int32)
        t = _gpu(k)
        B.bitonic_sort_segmented_keys(t, ot, asc, type_, max(lens) if bounded else 0)
        sort = (lambda a: O.sort_keys64(a.view(type_), i, asc).view(np.int64)) if i >= 3 else \
            (lambda a: O.sort_keys(a.view(type_), i, asc).view(np.int32))
        assert np.array_equal(t.cpu().numpy(), _oracle_segments(sort, k, off)), (type_, asc)


@pytest.mark.parametrize("lens", SEG_LENS, ids=["classes", "tiles", "supergroup"])
@pytest.mark.parametrize("values", ["index", "uniform", "mixed"])
def test_segment_pairs(lens, values):
    """Values in order in every segment, in none, and in every other one."""
    B = _bind()
    off = _segments(lens, 1)
    n = int(off[-1]) + 2
    k = _words("few", n, 31).astype(np.int32)
    v = W.uniform_i32(77, n)
    for s, (a, b) in enumerate(zip(off[:-1], off[1:])):
        if values == "index" or (values == "mixed" and s % 2 == 0):
            v[a:b] = np.arange(b - a, dtype=np.int32)
    kt, vt = _gpu(k), _gpu(v)
    B.bitonic_sort_segmented_pairs(kt, vt, torch.from_numpy(off).cuda(), False, "int32", max(lens))
    wk, wv = k.copy(), v.copy()
    for a, b in zip(off[:-1], off[1:]):
        wk[a:b], wv[a:b] = O.sort_pairs(k[a:b], v[a:b], 0, False)
    assert np.array_equal(kt.cpu().numpy(), wk)
    assert np.array_equal(vt.cpu().numpy(), wv)


def test_segments_without_a_bound_stay_with_the_network_below_its_limit():
    """No bound and no segment above 2^17 elements: the device leaves the big
    segments to the network's kernels."""
    B = _bind()
    lens = [1 << 17, 9000, 40_000, 100, (1 << 16) + 1]
    off = _segments(lens, 0)
    k = W.uniform_i32(3, int(off[-1]) + (1 << 21))   # the bound is the allocation's
    t = _gpu(k)
    B.bitonic_sort_segmented_i32(t, torch.from_numpy(off).cuda(), True)
    assert np.array_equal(t.cpu().numpy(), _oracle_segments(O.sort_i32, k, off))


@pytest.mark.parametrize("type_", ["int32", "float64"])
def test_segment_beyond_the_workspace(type_):
    """A segment with more elements than the workspace was laid out for (by
    the caller's bound) is sorted where it is; nothing is written past the
    workspace or the segment."""
    B = _bind()
    bound, n = (1 << 17) + 1, (1 << 17) + 300
    w = _words("uniform", n + 9, 8)
    k = w.astype(np.int32) if type_ == "int32" else w.copy()
    t = _gpu(k)
    B.bitonic_sort_segmented_keys(t, torch.tensor([0, n], device="cuda"), False, type_, bound)
    want = k.copy()
    want[:n] = O.sort_i32(k[:n], False) if type_ == "int32" else \
        O.sort_keys64(k[:n].view(type_), 5, False).view(np.int64)
    assert np.array_equal(t.cpu().numpy(), want)
