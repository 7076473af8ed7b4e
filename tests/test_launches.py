"""CPU test of how a map call's blocks are split into launches: each within the
32-bit work-items of a dispatch, together every block once, in order."""
import ctypes
import os

import pytest

from paper_1505_01120_amd import build as libbuild


@pytest.fixture(scope="module")
def launches():
    if not os.path.exists(libbuild.HOST_LIB):
        libbuild.build()
    f = ctypes.CDLL(libbuild.HOST_LIB).hl_launches
    U32, U64 = ctypes.c_uint32, ctypes.c_uint64
    f.argtypes, f.restype = [U64, U32, ctypes.POINTER(U64), ctypes.POINTER(U32), U64], U64

    def run(blocks, threads):
        first, count = (U64 * 64)(), (U32 * 64)()
        n = f(blocks, threads, first, count, 64)
        assert n <= 64
        return list(zip(first[:n], count[:n]))
    return run


@pytest.mark.parametrize("threads", [64, 256, 1024])
@pytest.mark.parametrize("units", [0, 1, 2, 5])
@pytest.mark.parametrize("off", [-1, 0, 1, 12345])
def test_launches(launches, threads, units, off):
    blocks = units * ((1 << 32) // threads) + off
    if blocks < 0:
        return
    at = 0
    for first, count in launches(blocks, threads):
        assert first == at and 0 < count * threads < 1 << 32
        at += count
    assert at == blocks
