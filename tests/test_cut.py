"""CPU tests of how calls are cut into tiles (the host logic that batched,
graph, chain and allocation-free reduces share)."""
import ctypes
import os

import pytest

import paper_1505_01120_amd as sc
from paper_1505_01120_amd import build as libbuild

CUS, OCC = 256, 4


@pytest.fixture(scope="module")
def cut():
    if not os.path.exists(libbuild.HOST_LIB):
        libbuild.build()
    lib = ctypes.CDLL(libbuild.HOST_LIB)
    U32 = ctypes.c_uint32
    lib.hl_tuning_defaults.argtypes, lib.hl_tuning_defaults.restype = [ctypes.POINTER(sc.Tuning)], None
    lib.hl_cut.argtypes = [ctypes.POINTER(sc.Tuning), ctypes.POINTER(sc.Tuning), U32, U32, U32,
                           ctypes.c_int, ctypes.POINTER(sc.Task), U32, U32, ctypes.POINTER(U32)]
    lib.hl_cut.restype = U32
    table = sc.Tuning()
    lib.hl_tuning_defaults(ctypes.byref(table))

    def f(tasks, mode=sc.BATCHED, per_cu=0, tuning=table, tuned=table, exec_blocks=0):
        tile = (U32 * len(tasks))()
        grid = lib.hl_cut(ctypes.byref(tuning), tuned and ctypes.byref(tuned), CUS, OCC,
                          exec_blocks, mode, (sc.Task * len(tasks))(*tasks), len(tasks), per_cu,
                          tile)
        return grid, list(tile)
    f.lib, f.table = lib, table
    return f


def task(kid, n):
    return sc.Task(kernel_id=kid, reduce_ops=sc.SUM, n=n, in0=4096, in1=8192)


@pytest.mark.parametrize("kid", [0, 4, 9, 10, 14, 20, 50, 100, 200, 1 << 20, 0xFFFFFFFF])
@pytest.mark.parametrize("n", [0, 1, 1000, 1 << 22, 1 << 40])
def test_unknown_kernel_ids(cut, kid, n):
    # the cut is made before the tasks are checked: an unknown id takes no
    # part in it, whatever stands around it
    for mode in (sc.PER_LAUNCH, sc.BATCHED, sc.GRAPH):
        for per_cu in (0, 2):
            cut([task(kid, n)], mode, per_cu)
            for other in (sc.POLY, sc.FMUL):
                good = [task(other, 300007)] * 3
                assert cut([task(kid, n)] + good, mode, per_cu) == \
                    (cut(good, mode, per_cu)[0], [0] + cut(good, mode, per_cu)[1]), (mode, per_cu)


def copy_of(t):
    return sc.Tuning.from_buffer_copy(bytes(t))


def test_callers_rows_are_the_cut(cut):
    small = [task(sc.FMUL, 300_000)] * 4
    assert cut(small)[0] and cut(small, tuning=copy_of(cut.table)) == cut(small)
    own = copy_of(cut.table)
    for mode in range(2):
        own.tile[mode][1][18] = 1 << 13
    assert cut(small, tuning=own) == (0, [1 << 13] * 4)
    # the rows that a tuner left are tuned rows as well, any other table's not
    assert cut(small, tuning=own, tuned=own)[0]
    assert not cut(small, tuned=own)[0] and not cut(small, tuned=None)[0]
    # rows that these calls do not read: batched, serving, Monte-Carlo
    other = copy_of(cut.table)
    other.tile[1][0][3] = other.tile[2][1][18] = other.tile[0][2][18] = 1 << 12
    assert cut(small, tuning=other) == cut(small)
    # enough work for the batched row, or Monte-Carlo tasks: the table
    assert not cut([task(sc.FMUL, 1 << 24)] * 64)[0]
    assert not cut(small + [sc.Task(kernel_id=sc.MC_PI, reduce_ops=sc.COUNT, n=1000)])[0]


def test_cache_file_carries_the_rule(cut, tmp_path):
    f = cut.lib.hl_tuning_small_by_time
    f.argtypes = [ctypes.c_char_p, ctypes.c_char_p, ctypes.POINTER(sc.Tuning), ctypes.c_int]
    f.restype = ctypes.c_int
    path = str(tmp_path / "t.json").encode()
    for arch, flag in ((b"a", 1), (b"b", 0), (b"a", 0), (b"b", 1)):
        assert f(path, arch, ctypes.byref(cut.table), flag) == flag
    # the library's own table is the autotuner's
    text = open(sc.sparkcl.TUNING_PATH).read()
    assert '"small_by_time": 1' in text


@pytest.mark.parametrize("block", [0, 256, 512, 1024])
@pytest.mark.parametrize("exec_blocks", [1, 2, 3, OCC, OCC + 1, 100])
def test_grid_is_resident(cut, block, exec_blocks):
    # the caller's blocks per CU count 256 threads and are clipped to what fits,
    # as for batches that the table cuts
    t = copy_of(cut.table)
    t.block[0] = t.block[1] = t.block_many = block
    for tasks in ([task(sc.FMUL, 300_000)] * 4, [task(sc.POLY, 5000), task(sc.FMUL, 5000)]):
        grid, _ = cut(tasks, tuning=t, exec_blocks=exec_blocks)
        assert grid == max(1, min(exec_blocks, OCC) * 256 // (block or 256)) * CUS
        assert cut(tasks, tuning=t)[0] == CUS
        assert cut(tasks, tuning=t, per_cu=3)[0] == 3 * CUS
