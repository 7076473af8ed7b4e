"""Small batches value by value: what a batch cut by estimated time writes
beside its sums, and blocking calls on both sides of the task count from which
a copy brings their results back, against the oracle."""
import numpy as np
import pytest
import torch

import datagen
import oracle
import paper_1505_01120_amd as sc
from gpu_helpers import DevParts, check_result, check_total, dev, oracle_result

pytestmark = pytest.mark.gpu

HOST_RESULTS = 384
ALL = datagen.SUM | datagen.MAX


@pytest.fixture(scope="module")
def ctx():
    c = sc.Context(device=0, arena_bytes=256 << 20)
    yield c
    c.destroy()


@pytest.mark.parametrize("count,n", [(1, 5), (1, 1 << 20), (3, 8786), (9, 131073), (48, 30007),
                                     (300, 4099), (16, 262147)])
@pytest.mark.parametrize("mode", [sc.BATCHED, sc.GRAPH])
@pytest.mark.parametrize("off", [0, 3])
def test_values_and_results(ctx, count, n, mode, off):
    parts = [datagen.make_part(datagen.FMUL if i % 3 else datagen.POLY, max(0, n - 7 * (i % 5)), i)
             for i in range(count)]
    tasks, bufs = [], []
    for i, p in enumerate(parts):
        x, y = dev(p.x, off), dev(p.y, (off + i) % 4) if p.y is not None else None
        buf = torch.full((p.n + 8,), float("nan"), device="cuda")
        tasks.append(sc.task(p.kid, p.n, x, y, buf[off:off + p.n], coef=p.coef, c=p.c))
        bufs.append((x, y, buf))
    per, total = ctx.reduce(tasks, mode)
    assert ctx.last_launch_shape()["tile_table"] == 0
    want = [oracle_result(p) for p in parts]
    for p, g, o, (_, _, buf) in zip(parts, per, want, bufs):
        check_result(g, o, p.kid, p.ops, f"kid={p.kid} n={p.n}")
        v = oracle.poly_map(p.x, p.coef) if p.kid == datagen.POLY else oracle.fmul_map(p.x, p.y)
        got = buf.cpu().numpy()
        assert np.array_equal(got[off:off + p.n].view(np.uint32), v.view(np.uint32)), (p.kid, p.n)
        assert np.isnan(got[:off]).all() and np.isnan(got[off + p.n:]).all()
    check_total(total, want, ALL)


@pytest.mark.parametrize("count", [HOST_RESULTS - 1, HOST_RESULTS, HOST_RESULTS + 1])
@pytest.mark.parametrize("mode", [sc.PER_LAUNCH, sc.BATCHED, sc.GRAPH])
def test_results_reach_the_host(ctx, count, mode):
    parts = [datagen.make_part(datagen.FMUL if i % 2 else datagen.POLY, 37 + i % 300, i)
             for i in range(count)]
    d = DevParts(parts)
    want = [oracle_result(p) for p in parts]
    for _ in range(2):
        per, total = ctx.reduce(d.tasks, mode)
        for p, g, o in zip(parts, per, want):
            check_result(g, o, p.kid, p.ops, f"n={p.n}")
        check_total(total, want, ALL)


@pytest.mark.parametrize("count", [5, HOST_RESULTS, HOST_RESULTS + 1])
def test_small_chains(ctx, count):
    stages = [(0.5, 2.0), (0.25, -1.0, 0.5)]
    parts = [datagen.make_part(datagen.FMUL if i % 2 else datagen.POLY, 4099 - i, i)
             for i in range(count)]
    d = DevParts(parts, 1, 2)
    per, total = ctx.reduce_chain(d.tasks, [sc.stage(s) for s in stages])
    want = []
    for p, g in zip(parts, per):
        v = oracle.chain_map(p.x, p.y, p.kid, p.coef, np.float32(p.c), stages)
        want.append(oracle.Result(sum=oracle.fsum(v), max=oracle.fmax(v), count=0, n=p.n))
        check_result(g, want[-1], p.kid, p.ops, f"n={p.n}")
    check_total(total, want, ALL)
