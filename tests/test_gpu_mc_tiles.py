"""Monte-Carlo batches on the executor instance of their own: counts equal to
the oracle's at the edges of its loop (1024 samples per iteration of a
256-thread block, odd last samples) and of its tiles, and equal to the
per-partition kernel's where the pair counter passes 2^32."""
import pytest

import datagen
import oracle
import paper_1505_01120_amd as sc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = sc.Context(device=0, arena_bytes=256 << 20)
    yield c
    c.destroy()


@pytest.mark.parametrize("n", [1, 2, 511, 512, 513, 1022, 1023, 1024, 1025, 1026, 2047, 2048, 2049,
                               131071, 131072, 131073, 132097, 1 << 23])
def test_loop_and_tile_edges(ctx, n):
    tasks = [sc.task(sc.MC_PI, n, seed=s, pid=p)
             for s, p in ((0, 0), (1, 7), ((1 << 63) + 12345, (1 << 32) - 1))]
    got = [r.count for r in ctx.map_partition(tasks, sc.BATCHED)]
    want = [oracle.run_task(datagen.MC_PI, datagen.COUNT, n, None, None, seed=t.seed,
                            pid=t.partition_id).count for t in tasks]
    assert got == want


def test_pair_counter_past_32_bits(ctx):
    n = (1 << 33) + (1 << 20) + 1
    task = [sc.task(sc.MC_PI, n, seed=5, pid=3)]
    batched = ctx.map_partition(task, sc.BATCHED)[0]
    single = ctx.map_partition(task, sc.PER_LAUNCH)[0]
    assert batched.count == single.count and batched.n == single.n == n
