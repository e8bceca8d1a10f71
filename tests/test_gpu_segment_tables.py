"""Segment tables at the sizes where the prep kernel reads them another way
and where the small segments change their kernel."""
import numpy as np
import pytest

from paper_1506_01446_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _bind():
    from paper_1506_01446_amd import binding as B
    return B


def _check(lens, type_, bound):
    B = _bind()
    wide = type_ == "int64"
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64) + 1
    n = int(off[-1])
    k = W.splitmix64(n, 0, n).view(np.int64) if wide else W.uniform_i32(n, n)
    t = torch.from_numpy(k.copy()).cuda()
    B.bitonic_sort_segmented_keys(t, torch.from_numpy(off).cuda(), True, type_, bound)
    want = k.copy()
    for a, b in zip(off[:-1], off[1:]):
        want[a:b].sort()
    assert np.array_equal(t.cpu().numpy(), want)


@pytest.mark.parametrize("nseg", [1, 1023, 1025, 2047, 2048, 2049, 3073, 8191, 8192, 8193, 9217])
def test_table_sizes(nseg):
    """Lengths of every class up to 14, with empty segments at the strides of
    the prep kernel's loads."""
    u = W.unit_doubles(nseg, nseg)
    lens = np.floor(2.0 ** (12.0 * u * u)).astype(np.int64)
    lens[::1024] = 0
    lens[-1] = 9000
    _check(lens, "int32", 9000)
    _check(lens, "int64", 1 << 16)


@pytest.mark.parametrize("type_", ["int32", "int64"])
@pytest.mark.parametrize("top", [6, 7, 9, 11, 12, 13])
def test_few_and_many_small_segments(type_, top):
    """One segment below and at the number from which on a launch holds many,
    full ones and lengths from one element on."""
    edge = 1 << ((22 if type_ == "int64" else 20) - top)
    for nseg in (edge - 1, edge, 3):
        if nseg << top > 1 << 22:
            continue
        lens = 1 + (W.splitmix64(top, 0, nseg) % np.uint64(1 << top)).astype(np.int64)
        lens[::3] = 1 << top
        _check(lens, type_, 1 << top)
