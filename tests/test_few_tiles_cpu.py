"""The tile programs of launches with few tiles (8 or 4 elements per thread)
and the 8-byte tile sorts with lane steps, on the CPU emulator of the
programs: each sorts, merges or finishes a phase of full and partial tiles,
and regroups that are synchronised per wave stay inside their waves."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_1506_01446_amd import workloads as W

HERE = os.path.dirname(os.path.abspath(__file__))

SORTS = [(L, 3, 4) for L in (9, 10, 11, 12)] + \
    [(10, 2, 6), (11, 3, 6), (12, 3, 6), (11, 4, 6), (12, 4, 6), (13, 4, 6)]
MERGES = [(11, 3, 1), (12, 3, 1), (11, 3, 3)]
PHASES = [(12, 3, 5), (13, 3, 5), (12, 3, 7)]


@pytest.fixture(scope="module")
def emu(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("emu") / "libemu.so")
    subprocess.run(["g++", "-O2", "-std=c++20", "-shared", "-fPIC", "-o", out,
                    os.path.join(HERE, "cpu_program_emulator.cpp")], check=True)
    lib = ctypes.CDLL(out)
    lib.emulate_tile.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_int,
                                 ctypes.POINTER(ctypes.c_int32), ctypes.c_uint32]
    lib.in_wave_regroups.argtypes = [ctypes.c_int] * 3 + [ctypes.POINTER(ctypes.c_int)]
    return lib


def _run(emu, L, r, kind, tile, valid):
    x = np.ascontiguousarray(tile, dtype=np.int32).copy()
    steps = emu.emulate_tile(L, r, kind, x.ctypes.data_as(ctypes.POINTER(ctypes.c_int32)), valid)
    assert steps >= 0, "program is not a permutation of the tile"
    return x, steps


@pytest.mark.parametrize("L,r,kind", SORTS)
def test_sorts(emu, L, r, kind):
    T = 1 << L
    for valid in (T, T - 1, T // 2 + 3, 2, 1):
        keys = W.uniform_i32(L * 17 + valid, T)
        out, steps = _run(emu, L, r, kind, keys, valid)
        assert steps == L * (L + 1) // 2
        assert (out[:valid] == np.sort(keys[:valid])).all()
        assert (out[valid:] == keys[valid:]).all()


@pytest.mark.parametrize("L,r,kind", MERGES)
def test_merges(emu, L, r, kind):
    T = 1 << L
    keys = W.uniform_i32(L, T)
    tile = np.concatenate([np.sort(keys[:T // 5]), np.sort(keys[T // 5:])[::-1]])
    out, steps = _run(emu, L, r, kind, tile, T)
    assert steps == L and (out == np.sort(keys)).all()


@pytest.mark.parametrize("L,r,kind", PHASES)
def test_phases(emu, L, r, kind):
    T = 1 << L
    for valid in (T, T - 1, T // 2 + 1, T // 2, 5):
        keys = W.uniform_i32(L + valid, T)
        keys[:min(valid, T // 2)].sort()
        if valid > T // 2:
            keys[T // 2:valid] = np.sort(keys[T // 2:valid])
        out, steps = _run(emu, L, r, kind, keys, valid)
        assert steps == L
        assert (out[:valid] == np.sort(keys[:valid])).all()
        assert (out[valid:] == keys[valid:]).all()


@pytest.mark.parametrize("L,r,kind", SORTS + MERGES + PHASES)
def test_in_wave_regroups(emu, L, r, kind):
    exact = ctypes.c_int()
    got = emu.in_wave_regroups(L, r, kind, ctypes.byref(exact))
    assert got >= 0, "a regroup synchronised per wave moves keys across waves"
    assert got == exact.value
