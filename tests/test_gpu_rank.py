"""The rank sorts of middle-sized single arrays against the CPU oracle, bit
for bit: every storage and key type, both directions, around each change of
tile and of the number of tiles, and ties within and across tiles."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1506_01446_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# Around the route's ends (2^11, 2^12; 2^16, 2^17), 16 tiles of each size, a
# tile of one element, a sample's edge (64) and a merging workgroup's (128).
SIZES = sorted({(1 << k) + d for k in range(11, 18) for d in (-1, 0, 1)} |
               {5 * 1024 + 1, 9 * 512 - 1, 17 * 1024 + 64, 3 * 4096 + 65, 20_000, 16 * 4096 + 127,
                17 * 4096, 31 * 4096 + 1, 100_003})


def _gpu(a):
    return torch.from_numpy(a.copy()).cuda()


def _words(n, seed, kind):
    w = W.splitmix64(seed, 0, n).view(np.int64)
    if kind == "few":        # runs of ties longer than a sample and a tile
        return w[(W.splitmix64(seed + 1, 0, n) >> np.uint64(62)).astype(np.int64)]
    if kind == "extremes":   # padding's own value and its opposite
        return np.where(w & 64, np.int64(2**63 - 1), np.int64(-2**63))
    if kind == "sorted":
        return np.sort(w)
    if kind == "reverse":
        return np.sort(w)[::-1].copy()
    return w


KINDS = ["uniform", "few", "extremes", "sorted", "reverse"]


@pytest.mark.parametrize("n", SIZES)
def test_rank_sorts(n):
    from paper_1506_01446_amd import binding as B
    for i, kind in enumerate(KINDS):
        asc = (i + n) % 2 == 0
        w = _words(n, n + i, kind)
        t32, t64 = ["int32", "uint32", "float32"][(i + n) % 3], ["int64", "uint64", "float64"][i % 3]
        k = (w >> 32).astype(np.int32)
        if kind == "extremes":
            k = np.where(w < 0, np.int32(-2**31), np.int32(2**31 - 1))
        t = _gpu(k)
        B.bitonic_sort_keys(t, asc, t32)
        want = O.sort_keys(k.view(t32), (i + n) % 3, asc).view(np.int32)
        assert np.array_equal(t.cpu().numpy(), want), (kind, t32)
        t = _gpu(w)
        B.bitonic_sort_keys64(t, asc, t64)
        want = O.sort_keys64(w.view(t64), 3 + i % 3, asc).view(np.int64)
        assert np.array_equal(t.cpu().numpy(), want), (kind, t64)
        v = np.arange(n, dtype=np.int32) if i % 2 else W.uniform_i32(n + 3, n) >> 31
        kt, vt = _gpu(k), _gpu(v)
        B.bitonic_sort_pairs(kt, vt, asc, t32)
        wk, wv = O.sort_pairs(k.view(t32), v, (i + n) % 3, asc)
        assert np.array_equal(kt.cpu().numpy(), wk.view(np.int32)), (kind, t32)
        assert np.array_equal(vt.cpu().numpy(), wv), (kind, t32)


def test_neighbours_are_untouched():
    """Arrays off a 16-byte boundary inside a larger one."""
    from paper_1506_01446_amd import binding as B
    for n in (5001, 30_000, 65_537):
        k = W.uniform_i32(n, n + 6)
        t = _gpu(k)
        B.bitonic_sort_i32(t[3:3 + n], False)
        want = k.copy()
        want[3:3 + n] = O.sort_i32(k[3:3 + n], False)
        assert np.array_equal(t.cpu().numpy(), want)


def test_captured_stream_runs_the_network():
    """A captured sort takes no workspace (it is the network) and sorts new
    keys at each replay, with eager sorts between."""
    from paper_1506_01446_amd import binding as B
    n = 30_001
    buf = torch.empty(n, dtype=torch.int32, device="cuda")
    eager = torch.empty_like(buf)
    B.bitonic_sort_i32(buf, True)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        B.bitonic_sort_i32(buf, True)
    for r in range(3):
        k = W.uniform_i32(r, n)
        buf.copy_(torch.from_numpy(k))
        eager.copy_(torch.from_numpy(k))
        g.replay()
        B.bitonic_sort_i32(eager, True)
        torch.cuda.synchronize()
        want = O.sort_i32(k, True)
        assert np.array_equal(buf.cpu().numpy(), want), r
        assert np.array_equal(eager.cpu().numpy(), want), r
