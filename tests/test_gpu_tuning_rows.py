"""Whose per-launch rows are in force decides how a small batch is cut: a table
read and set again changes nothing, rows that the caller changed are the cut
until they are changed back, and a tuned context and one that loads its cache
file cut alike."""
import json

import pytest
import torch

import paper_1505_01120_amd as sc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tasks():
    x = torch.randn(8, 300_000, device="cuda")
    return [sc.task(sc.FMUL, 300_000, x[i], x[i + 4], c=0.5) for i in range(4)], x


def cut(ctx, tasks):
    per, total = ctx.reduce(tasks[0], sc.BATCHED)
    return ctx.last_launch_shape(), [r.sum for r in per], total.sum


def test_set_tuning(tasks):
    with sc.Context(device=0, arena_bytes=64 << 20) as ctx:
        first, table = cut(ctx, tasks), ctx.get_tuning()
        ctx.set_tuning(table)
        assert cut(ctx, tasks) == first
        kept = table.tile[0][1][18]
        table.tile[0][1][18] = 1 << 10
        ctx.set_tuning(table)
        assert cut(ctx, tasks)[0]["ntiles"] == 4 * -(-300_000 // 1024) != first[0]["ntiles"]
        table.tile[0][1][18] = kept
        ctx.set_tuning(table)
        assert cut(ctx, tasks) == first


def test_cache_files(tasks, tmp_path):
    with sc.Context(device=0, arena_bytes=64 << 20) as ctx:
        first = cut(ctx, tasks)
    table = json.load(open(sc.sparkcl.TUNING_PATH))
    rows = next(iter(table.values()))["tile"]["per_launch"]["fmul"]
    for entry in table.values():
        del entry["small_by_time"]  # a table that the caller wrote
    path = tmp_path / "own.json"
    path.write_text(json.dumps(table))
    with sc.Context(device=0, arena_bytes=64 << 20, tune_cache=str(path)) as ctx:
        assert cut(ctx, tasks)[0]["ntiles"] == 4 * -(-300_000 // rows[18]) != first[0]["ntiles"]


def test_autotuned(tasks, tmp_path):
    path = str(tmp_path / "tuned.json")
    with sc.Context(device=0, arena_bytes=3 << 30) as ctx:
        with pytest.raises(sc.SparkclError):
            ctx.autotune(12, 5)  # refused: nothing changes
        before = cut(ctx, tasks)
        ctx.autotune(18, 18, path)
        tuned = cut(ctx, tasks)
    assert tuned[0]["ntiles"] == before[0]["ntiles"]
    with sc.Context(device=0, arena_bytes=64 << 20, tune_cache=path) as ctx:
        loaded = cut(ctx, tasks)
    assert loaded == tuned


@pytest.mark.parametrize("block", [256, 1024])
def test_callers_blocks_per_cu(block):
    # a small batch runs on no more blocks than a large one, which the table cuts
    x = torch.rand(1 << 26, device="cuda")
    large = [sc.task(sc.POLY, 1 << 20, x[i << 20:], coef=(1.0, 2.0)) for i in range(64)]
    small = [sc.task(sc.POLY, 1 << 20, x[i << 20:], coef=(1.0, 2.0)) for i in range(3)]
    with sc.Context(device=0, arena_bytes=64 << 20, exec_blocks_per_cu=100) as ctx:
        t = ctx.get_tuning()
        t.block[0] = block
        for b in range(sc.TUNE_BUCKETS):
            t.tile[1][0][b] = 1 << 13  # batched
        ctx.set_tuning(t)
        ctx.reduce(large, sc.BATCHED)
        most = ctx.last_launch_shape()
        assert most["tile_table"] == 1 and most["ntiles"] > most["grid"]
        want, _ = ctx.reduce(small, sc.PER_LAUNCH)
        got, _ = ctx.reduce(small, sc.BATCHED)
        shape = ctx.last_launch_shape()
        assert shape["tile_table"] == 0 and shape["grid"] <= most["grid"]
        for g, w in zip(got, want):
            assert abs(g.sum - w.sum) <= 1e-9 * w.sum and g.max == w.max
