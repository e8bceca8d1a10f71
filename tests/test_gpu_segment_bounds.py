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


# Segments for the network (up to class 16, of 8-byte elements 17), for the digits (above)
# and for neither (2^13 and below), with the long ones first, last and
# between; "many" has enough of the middle classes for the network to keep
# them beside the digits' launches, "few" has not, "none" has no long one.
TABLES = {
    "many": [(1 << 18) + 1, 0, 9000] + [1 << 16] * 30 + [(1 << 17) + 1, 1 << 17, 8192, 3] +
            [40_001] * 9 + [1 << 14, 8193, 300_000],
    "few": [8193, (1 << 19) + 77, 1 << 17, 100, (1 << 14) + 1, 0, 1 << 18],
    "none": [1 << 17, 9000, 40_000, 100, (1 << 16) + 1, 0, 8193, 1 << 14],
    "long": [1 << 18, (1 << 17) + 1],
}


@pytest.mark.parametrize("table", list(TABLES))
@pytest.mark.parametrize("bound_log2", [20, 25])
def test_each_segment_by_its_own_class(table, bound_log2):
    B = _bind()
    lens = TABLES[table]
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64) + 5
    n = int(off[-1]) + 3
    ot = torch.from_numpy(off).cuda()
    arena = 1 << 22    # the table lies in a larger allocation
    for i, type_ in enumerate(["int32", "uint32", "float32", "int64", "uint64", "float64"]):
        asc = (i + bound_log2) % 2 == 0
        w = W.splitmix64(9 + i, 0, n).view(np.int64)
        k = w if i >= 3 else w.astype(np.int32)
        t = torch.empty(arena, dtype=torch.int64 if i >= 3 else torch.int32, device="cuda")[:n]
        t.copy_(torch.from_numpy(k.copy()))
        B.bitonic_sort_segmented_keys(t, ot, asc, type_, 1 << bound_log2)
        want = k.copy()
        for a, b in zip(off[:-1], off[1:]):
            want[a:b] = O.sort_keys64(k[a:b].view(type_), i, asc).view(np.int64) if i >= 3 else \
                O.sort_keys(k[a:b].view(type_), i, asc).view(np.int32)
        assert np.array_equal(t.cpu().numpy(), want), (type_, asc)


@pytest.mark.parametrize("table", list(TABLES))
@pytest.mark.parametrize("ordered", [True, False])
def test_each_segment_by_its_own_class_pairs(table, ordered):
    B = _bind()
    lens = TABLES[table]
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    n = int(off[-1])
    k = (W.uniform_i32(4, n) >> 20).astype(np.int32)      # many ties
    v = np.arange(n, dtype=np.int32) if ordered else W.uniform_i32(5, n)
    kt = torch.empty(1 << 22, dtype=torch.int32, device="cuda")[:n]
    vt = torch.empty_like(kt)
    kt.copy_(torch.from_numpy(k))
    vt.copy_(torch.from_numpy(v))
    B.bitonic_sort_segmented_pairs(kt, vt, torch.from_numpy(off).cuda(), True, "int32", 1 << 21)
    for a, b in zip(off[:-1], off[1:]):
        k[a:b], v[a:b] = O.sort_pairs(k[a:b], v[a:b], 0, True)
    assert np.array_equal(kt.cpu().numpy(), k)
    assert np.array_equal(vt.cpu().numpy(), v)


def test_refused_table_touches_no_key():
    """With validation on, a table with a segment above its bound leaves the
    keys alone on this route too."""
    B = _bind()
    k = W.uniform_i32(6, 2_000_000)
    t = torch.from_numpy(k.copy()).cuda()
    off = torch.tensor([0, 300_000, 2_000_000], device="cuda")
    B.bitonic_set_tuning_value("validate", 1)
    try:
        B.bitonic_validation_error()
        B.bitonic_sort_segmented_keys(t, off, True, "int32", 1 << 20)
        assert B.bitonic_validation_error() == 3
        assert np.array_equal(t.cpu().numpy(), k)
    finally:
        B.bitonic_set_tuning_value("validate", 0)


@pytest.mark.parametrize("total", ["unknown", "exact", "too small"])
@pytest.mark.parametrize("bounded", [True, False])
def test_total_of_all_segments(total, bounded):
    """The C entry with a bound on all segments' elements: it sizes the
    workspace; one that the table exceeds costs time only."""
    B = _bind()
    lens = [700_001, 0, 9000, 64]
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64) + 11
    n = int(off[-1])
    k = W.uniform_i32(8, n)
    t = torch.empty(1 << 22, dtype=torch.int32, device="cuda")
    t[:n].copy_(torch.from_numpy(k))
    ot = torch.from_numpy(off).cuda()
    rc = B.load().bitonic_sort_segmented_within(
        t.data_ptr(), None, ot.data_ptr(), len(lens), (1 << 20) if bounded else 0,
        {"unknown": 0, "exact": n - 11, "too small": 600_000}[total], 0, 1,
        torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    for a, b in zip(off[:-1], off[1:]):
        k[a:b] = np.sort(k[a:b])
    assert np.array_equal(t[:n].cpu().numpy(), k)
    assert B.load().bitonic_sort_segmented_within(
        t.data_ptr(), None, ot.data_ptr(), len(lens), 1 << 20, -1, 0, 1, None) == -1


# Around the tiles (2^14 4-byte, 2^13 8-byte elements), a group of 16 and a
# supergroup of 256 of them.
TILES = {
    "classes": [(1 << 17) + 1, 0, 8193, 5, 8192, 1 << 14, (1 << 14) + 1, 70_001],
    "tiles": [1 << 18, 1, (1 << 18) + 1, 3 * 8192, 300, 0, 150_000],
    "supergroup": [(1 << 21) + 8193, 20_000, 1 << 17],
}


@pytest.mark.parametrize("lens", list(TILES.values()), ids=list(TILES))
def test_segments_by_digits(lens):
    """With room for more elements than there are, tables of fewer than 2^19
    elements go by digits too."""
    B = _bind()
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64) + 3
    n = int(off[-1]) + 5
    ot = torch.from_numpy(off).cuda()
    st = torch.cuda.current_stream().cuda_stream
    for i, type_ in enumerate(["int32", "uint32", "float32", "int64", "uint64", "float64"]):
        for kind in ("uniform", "few"):
            asc = (i % 2 == 0) == (kind == "few")
            w = W.splitmix64(70 + i, 0, n).view(np.int64)
            if kind == "few":
                w = w & np.int64(0x0000FF000000FF00)
            k = w.copy() if i >= 3 else w.astype(np.int32)
            t = torch.from_numpy(k.copy()).cuda()
            assert B.load().bitonic_sort_segmented_within(
                t.data_ptr(), None, ot.data_ptr(), len(lens), 1 << 22, 1 << 22, i, int(asc),
                st) == 0
            for a, b in zip(off[:-1], off[1:]):
                k[a:b] = O.sort_keys64(k[a:b].view(type_), i, asc).view(np.int64) if i >= 3 else \
                    O.sort_keys(k[a:b].view(type_), i, asc).view(np.int32)
            assert np.array_equal(t.cpu().numpy(), k), (type_, kind, asc)
    k = (W.uniform_i32(31, n) >> 22).astype(np.int32)
    v = W.uniform_i32(77, n)
    for s, (a, b) in enumerate(zip(off[:-1], off[1:])):
        if s % 2 == 0:    # in order in every other segment
            v[a:b] = np.arange(b - a, dtype=np.int32)
    kt, vt = torch.from_numpy(k.copy()).cuda(), torch.from_numpy(v.copy()).cuda()
    assert B.load().bitonic_sort_segmented_within(
        kt.data_ptr(), vt.data_ptr(), ot.data_ptr(), len(lens), 1 << 22, 1 << 22, 0, 0, st) == 0
    for a, b in zip(off[:-1], off[1:]):
        k[a:b], v[a:b] = O.sort_pairs(k[a:b], v[a:b], 0, False)
    assert np.array_equal(kt.cpu().numpy(), k)
    assert np.array_equal(vt.cpu().numpy(), v)
