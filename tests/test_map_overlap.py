"""CPU test of the check that decides whether a map call's tasks run in one
launch: against all pairs of arrays, byte by byte of their ranges."""
import ctypes
import os
import random

import pytest

import paper_1505_01120_amd as sc
from paper_1505_01120_amd import build as libbuild


@pytest.fixture(scope="module")
def independent():
    if not os.path.exists(libbuild.HOST_LIB):
        libbuild.build()
    f = ctypes.CDLL(libbuild.HOST_LIB).hl_tasks_independent
    f.argtypes, f.restype = [ctypes.POINTER(sc.Task), ctypes.c_uint32], ctypes.c_int
    return lambda tasks: bool(f((sc.Task * max(len(tasks), 1))(*tasks), len(tasks)))


def all_pairs(tasks):
    ranges = []
    for i, t in enumerate(tasks):
        arrays = [(t.in0, False), (t.in1 if t.kernel_id == sc.FMUL else None, False), (t.out, True)]
        ranges += [(a, a + 4 * t.n, i, w) for a, w in arrays if a and t.n]
    return not any(p[2] != q[2] and (p[3] or q[3]) and p[0] < q[1] and q[0] < p[1]
                   for p in ranges for q in ranges)


def test_known_orders(independent):
    def poly(x, out, n=100):
        return sc.task(sc.POLY, n, x=x, out=out, coef=(1.0, 2.0))
    assert independent([])
    assert independent([poly(4096, 8192), poly(4096, 12288)])        # a shared input
    assert independent([poly(4096, 4096), poly(8192, 8192)])         # in place
    assert independent([poly(4096, 8192), poly(4496, 8592)])         # adjacent
    assert not independent([poly(4096, 8192), poly(8192, 12288)])    # a pipeline
    assert not independent([poly(4096, 8192), poly(12288, 8588)])    # one float of output
    assert not independent([poly(4096, 8192, 1000), poly(16384, 4100, 1)])
    assert independent([poly(4096, 8192), poly(8192, 12288, 0)])     # nothing to do


@pytest.mark.parametrize("seed", range(8))
def test_random_tasks_against_all_pairs(independent, seed):
    rng = random.Random(seed)
    seen = set()
    for _ in range(400):
        span = rng.choice((200, 2000, 20000))
        tasks = []
        for _ in range(rng.randint(1, 8)):
            at = [4 * rng.randint(1, span) for _ in range(3)]
            if rng.random() < 0.3:
                at[2] = at[0]
            tasks.append(sc.task(rng.choice((sc.POLY, sc.FMUL)), rng.randint(0, 60), x=at[0],
                                 y=at[1], out=at[2], coef=(1.0,)))
        want = all_pairs(tasks)
        seen.add(want)
        assert independent(tasks) == want, [(t.in0, t.in1, t.out, t.n) for t in tasks]
    assert seen == {True, False}
