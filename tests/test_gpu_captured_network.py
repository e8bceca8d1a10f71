"""The network on uint32 and float32 keys of every size: the plain calls run it
on a stream that is being captured (elsewhere they sort longer arrays by rank
or digits, and plans exist for int32 and the 8-byte sorts only)."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1506_01446_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_1506_01446_amd import binding as B  # noqa: E402

TYPES = {"uint32": (O.KEY_U32, np.uint32), "float32": (O.KEY_F32, np.float32)}
# NaNs of both signs, infinities, zeros, denormals
SPECIAL = np.array([0x7FC00001, 0xFFC00001, 0x7F800000, 0xFF800000, 0, 0x80000000, 1, 0x80000001,
                    0x7FFFFFFF, 0xFFFFFFFF], dtype=np.uint32)
CANARY = np.int32(0x5AFE5AFE)


def _check(n, type_, asc, shift=0, replays=2):
    kt, dt = TYPES[type_]
    buf = torch.full((n + 8,), int(CANARY), dtype=torch.int32, device="cuda")
    view = buf[shift:shift + n]
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        B.bitonic_sort_keys(view, asc, type_)
    for r in range(replays):
        bits = W.uniform_i32(n + 7 * r, n).view(np.uint32).copy()
        bits[: len(SPECIAL)] = SPECIAL
        view.copy_(torch.from_numpy(bits.view(np.int32).copy()))
        g.replay()
        torch.cuda.synchronize()
        h = buf.cpu().numpy()
        assert (h[:shift] == CANARY).all() and (h[shift + n:] == CANARY).all()
        want = O.sort_keys(bits.view(dt), kt, asc).view(np.int32)
        assert np.array_equal(h[shift:shift + n], want), (n, type_, asc, shift, r)


@pytest.fixture
def tuned():
    """Sets tuning values for the test."""
    saved = {}

    def set_(name, value):
        saved.setdefault(name, B.bitonic_get_tuning_value(name))
        B.bitonic_set_tuning_value(name, value)

    yield set_
    for name, value in saved.items():
        B.bitonic_set_tuning_value(name, value)


@pytest.mark.parametrize("type_", list(TYPES))
@pytest.mark.parametrize("n", [4097, 8192, 8193, 70_001, 1 << 17, (1 << 20) + 3])
def test_sizes_and_alignments(n, type_):
    for shift in (0, 1, 2, 3):
        _check(n, type_, (n + shift) % 2 == 0, shift)
    _check(n, type_, (n + 1) % 2 == 0)


@pytest.mark.parametrize("asc", [True, False])
def test_looping_merge_decodes_floats(tuned, asc):
    """One looping workgroup per compute unit; and no workspace is taken."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    n = ((2 * cus) << 14) + 999
    tuned("merge_blocks_per_cu", 1)
    B.bitonic_release_workspaces()
    _check(n, "float32", asc)
    before = torch.cuda.mem_get_info()[0]
    B.bitonic_release_workspaces()
    assert torch.cuda.mem_get_info()[0] < before + 4 * n


@pytest.mark.parametrize("type_", list(TYPES))
@pytest.mark.parametrize("t", [11, 12, 13, 14])
def test_phase_merge_decodes(tuned, t, type_):
    """Phase t + 1 as the last launch, and followed by further phases."""
    tuned("tile_log2", t)
    for on in (1, 0):
        tuned("phase_merge", on)
        for n in (1 << (t + 1), (1 << (t + 1)) - 3, (1 << (t + 3)) + 4099):
            for asc in (True, False):
                _check(n, type_, asc)


@pytest.mark.parametrize("sort_tile", [14, 15])
def test_larger_tile_sorts_decode(tuned, sort_tile):
    tuned("tile_log2", 13)
    tuned("sort_tile_log2", sort_tile)
    for type_ in TYPES:
        for k in (sort_tile, sort_tile + 1, 18):
            _check(1 << k, type_, k % 2 == 0)
