"""Short single arrays (one to 64 tiles, fewer elements per thread) against the
CPU oracle: every storage, both directions, around each tile's size."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1506_01446_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SIZES = sorted({2, 3, 100} | {(1 << k) + d for k in range(9, 17) for d in (-1, 0, 1)} | {50_000})


def _gpu(a):
    return torch.from_numpy(a.copy()).cuda()


@pytest.mark.parametrize("n", SIZES)
def test_short_arrays(n):
    from paper_1506_01446_amd import binding as B
    for i, type_ in enumerate(["int32", "uint32", "float32"]):
        asc = (i + n) % 2 == 0
        k = W.uniform_i32(n + i, n)
        v = W.uniform_i32(n + 7, n) >> 30
        t = _gpu(k)
        B.bitonic_sort_keys(t, asc, type_)
        assert np.array_equal(t.cpu().numpy(), O.sort_keys(k.view(type_), i, asc).view(np.int32))
        t, vt = _gpu(k >> 22 if type_ != "float32" else k), _gpu(v)
        kk = t.cpu().numpy()
        B.bitonic_sort_pairs(t, vt, asc, type_)
        wk, wv = O.sort_pairs(kk.view(type_), v, i, asc)
        assert np.array_equal(t.cpu().numpy(), wk.view(np.int32))
        assert np.array_equal(vt.cpu().numpy(), wv)
    for i, type_ in enumerate(["int64", "uint64", "float64"]):
        k = W.uniform_i64(n + i, n)
        if i == 0:
            k = k >> 60     # many ties on the high word
        t = _gpu(k)
        B.bitonic_sort_keys64(t, i % 2 == 0, type_)
        want = O.sort_keys64(k.view(type_), 3 + i, i % 2 == 0).view(np.int64)
        assert np.array_equal(t.cpu().numpy(), want), type_
