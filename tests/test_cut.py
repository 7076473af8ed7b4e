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
    lib.hl_cut.argtypes = [ctypes.POINTER(sc.Tuning), U32, U32, ctypes.c_int,
                           ctypes.POINTER(sc.Task), U32, U32, ctypes.POINTER(U32)]
    lib.hl_cut.restype = ctypes.c_int
    table = sc.Tuning()
    lib.hl_tuning_defaults(ctypes.byref(table))

    def f(tasks, mode=sc.BATCHED, per_cu=0, tuning=table):
        tile = (U32 * len(tasks))()
        by_time = lib.hl_cut(ctypes.byref(tuning), CUS, OCC, mode, (sc.Task * len(tasks))(*tasks),
                             len(tasks), per_cu, tile)
        return bool(by_time), list(tile)
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
