"""Blocking calls' results, which the launch writes to the host up to 1024 tasks
and a copy brings back beyond: every field the same as the asynchronous call's,
over the modes, with growing and shrinking calls on one context and chains and
Monte-Carlo batches between them."""
import numpy as np
import pytest
import torch

import datagen
import paper_1505_01120_amd as sc
from gpu_helpers import DevParts, check_result, oracle_result

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = sc.Context(device=0, arena_bytes=256 << 20)
    yield c
    c.destroy()


@pytest.mark.parametrize("mode", [sc.PER_LAUNCH, sc.BATCHED, sc.GRAPH])
@pytest.mark.parametrize("count", [1, 40, 1023, 1024, 1025, 2])
def test_blocking_equals_async(ctx, mode, count):
    if mode == sc.PER_LAUNCH and count > 40:
        pytest.skip("one launch per task")
    parts = [datagen.make_part(datagen.FMUL if i % 2 else datagen.POLY, 37 + i % 300, i)
             for i in range(count)]
    d = DevParts(parts)
    res = torch.zeros(64 * count, dtype=torch.uint8, device="cuda")
    tot = torch.zeros(64, dtype=torch.uint8, device="cuda")
    ctx.reduce_async(d.tasks, mode, res, tot)
    torch.cuda.synchronize()
    s = res.view(torch.float64).view(-1, 8)[:, 0].cpu().tolist()
    m = res.view(torch.float32).view(-1, 16)[:, 2].cpu().tolist()
    for _ in range(3):
        per, total = ctx.reduce(d.tasks, mode)
        assert [g.sum for g in per] == s and [g.max for g in per] == m
        assert total.sum == tot.view(torch.float64)[0].item()
        assert total.n == sum(p.n for p in parts) and all(g.t_done_ns for g in per)
    for p, g in list(zip(parts, per))[::97]:
        check_result(g, oracle_result(p), p.kid, p.ops, f"n={p.n}")
    assert ctx.last_kernel_ms() > 0


def test_other_blocking_calls(ctx):
    mc = [datagen.make_part(datagen.MC_PI, 5001 + i, i, with_data=False) for i in range(70)]
    for _ in range(2):
        for p, g in zip(mc, ctx.map_partition(DevParts(mc).tasks)):
            check_result(g, oracle_result(p), p.kid, p.ops, f"n={p.n}")
    parts = [datagen.make_part(datagen.POLY, 4099, i) for i in range(5)]
    d = DevParts(parts)
    per, total = ctx.reduce_chain(d.tasks, [sc.stage((0.5, 2.0))])
    plain, _ = ctx.reduce(d.tasks, sc.BATCHED)
    for g, p in zip(per, plain):
        assert g.n == p.n and abs(g.sum - (0.5 * p.n + 2.0 * p.sum)) <= 1e-3 * (p.n + abs(p.sum))
    assert total.n == 5 * 4099
