"""Segmented sorts whose bound on the segment length is far above their
segments: the bound may be any number from the longest segment's length on."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1506_01446_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _bind():
    from paper_1506_01446_amd import binding as B
    return B


def _tail(n, dtype):
    """n elements at the very end of an allocation of 16 MiB."""
    torch.cuda.empty_cache()
    size = torch.empty(0, dtype=dtype).element_size()
    return torch.empty((16 << 20) // size, dtype=dtype, device="cuda")[-n:]


@pytest.mark.parametrize("bound_log2", [18, 21, 23, 31])
@pytest.mark.parametrize("lens", [[1000], [8191], [200, 0, 700, 1], [3000, 2000, 3191]])
@pytest.mark.parametrize("type_", ["int32", "float64"])
def test_small_arrays_with_loose_bounds(type_, lens, bound_log2):
    """Fewer elements than one big segment's, in all and up to the end of
    their allocation: there is nothing to lay a digit workspace out for."""
    B = _bind()
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    n = int(off[-1])
    wide = type_ == "float64"
    k = W.splitmix64(n + bound_log2, 0, n).view(np.int64) if wide else W.uniform_i32(n, n)
    t = _tail(n, torch.int64 if wide else torch.int32)
    t.copy_(torch.from_numpy(k.copy()))
    B.bitonic_sort_segmented_keys(t, torch.from_numpy(off).cuda(), False, type_, 1 << bound_log2)
    want = k.copy()
    for a, b in zip(off[:-1], off[1:]):
        want[a:b] = O.sort_keys64(k[a:b].view(type_), 5, False).view(np.int64) if wide else \
            O.sort_i32(k[a:b], False)
    assert np.array_equal(t.cpu().numpy(), want)
