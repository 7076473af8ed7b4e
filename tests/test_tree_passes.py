"""CPU tests of how an array reduce is split into passes: chunks that the
kernels take, a tree that ends in one row, and scratch that does not grow with
the input."""
import ctypes
import os
import random

import pytest

from paper_1505_01120_amd import build as libbuild

CUS = 256
MIB = 1 << 20


@pytest.fixture(scope="module")
def passes():
    if not os.path.exists(libbuild.HOST_LIB):
        libbuild.build()
    f = ctypes.CDLL(libbuild.HOST_LIB).hl_tree_passes
    U32 = ctypes.c_uint32
    f.argtypes = [U32, ctypes.c_uint64, U32, ctypes.c_int, ctypes.POINTER(U32 * 7), U32]
    f.restype = U32
    names = ("count", "chunk", "rows", "cpt", "threads", "groups", "cols")

    def run(k, length, least=False):
        out = (U32 * 7 * 64)()
        n = f(k, length, CUS, int(least), out, 64)
        assert n <= 64
        return [dict(zip(names, p)) for p in out[:n]]
    return run


def scratch(plan, length):
    """Bytes of the two buffers that the passes' rows alternate in."""
    return sum(p["rows"] * length * 4 for p in plan[:-1][:2])


def in_columns(k, length, vector):
    """Scratch when every pass folds whole columns (of four floats or one) in
    chunks of up to 4096 leaves that fill the GPU."""
    total, count, n = 0, k, 0
    blocks, target = -(-length // (256 * vector)), 4 * CUS
    while True:
        chunk = None
        if vector == 4:
            ch = min(count, 64)
            nch = -(-count // ch)
            if nch <= 64 and (-(-(length // 4) // 2048) * nch >= 2 * CUS or any(
                    -(-(length // 4) // (256 * c)) * nch >= target // 2 for c in (4, 2))):
                chunk = ch
        if chunk is None:
            if count <= 4096 and (blocks >= target or count <= 64):
                chunk = count
            else:
                chunk = 1 << (max(1, count * blocks // target).bit_length() - 1)
                chunk = min(max(chunk, 8), 4096)
                while -(-count // chunk) > 65535:
                    chunk *= 2
                chunk = min(chunk, count)
        rows = -(-count // chunk)
        if rows == 1:
            return total
        if n < 2:
            total += rows * length * 4
        count, n = rows, n + 1


def shapes():
    rng = random.Random(7)
    yield from [(1, 1), (2, 3), (1 << 24, 1), (1 << 24, 3), (1 << 24, 4), (1 << 24, 256),
                (1 << 20, 4096), (1 << 20, 4097), (65536, 4096), (1 << 18, 3000), (1 << 18, 2049),
                (131072, 2047), (1 << 20, 1024), (48, 1000003), (64, 1 << 22), (4096, 1 << 22)]
    for _ in range(4000):
        length = int(2 ** rng.uniform(0, 24))
        yield max(1, int(2 ** rng.uniform(0, min(24, 36 - length.bit_length())))), length


def test_passes(passes):
    for k, length in shapes():
        for least in (False, True):
            plan = passes(k, length, least)
            count = k
            for p in plan:
                assert p["count"] == count and p["rows"] == -(-count // p["chunk"]), (k, length, p)
                assert p["rows"] == 1 or p["chunk"] & (p["chunk"] - 1) == 0, (k, length, p)
                if p["groups"]:
                    per = p["chunk"] // p["groups"]
                    assert p["chunk"] == per * p["groups"] and per & (per - 1) == 0 and per <= 64
                    assert p["cols"] * p["groups"] <= p["threads"] <= 1024
                    assert p["threads"] % 64 == 0
                else:
                    assert length >= 4 and p["chunk"] <= (64 if p["cpt"] > 1 else 4096)
                    assert p["rows"] <= 65535
                count = p["rows"]
            assert count == 1


def test_scratch_is_bounded(passes):
    for k, length in shapes():
        vector = 1 if length % 4 else 4
        before = in_columns(k, length, vector)
        # no more than columns take (floats of four), or 8 MiB a pass
        most = max(in_columns(k, length, 4), before, 2 * 8 * MIB)
        plan = passes(k, length)
        assert scratch(plan, length) <= most, (k, length, scratch(plan, length), most)
        if length >= 4:
            assert scratch(passes(k, length, True), length) <= before, (k, length)
    for k, length in ((1 << 20, 4096), (65536, 4096), (1 << 18, 3000)):
        assert scratch(passes(k, length), length) <= 7 * MIB, (k, length)
