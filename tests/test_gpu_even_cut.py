"""Batches of streaming tasks that are cut by estimated time: tile sizes at the
ends of the rule's range (one tile per task, about two per block, values written
beside the sums), against the oracle in both batched modes, and the
allocation-free call bit for bit the same."""
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


@pytest.mark.parametrize("count,n", [(1, 5), (3, 8786), (9, 131073), (48, 30007), (300, 4099),
                                     (16, 262147), (4, (1 << 21) + 3)])
@pytest.mark.parametrize("out", [False, True])
def test_even_cut(ctx, count, n, out):
    parts = [datagen.make_part(datagen.FMUL if i % 3 else datagen.POLY, max(0, n - 7 * (i % 5)), i)
             for i in range(count)]
    d = DevParts(parts, 1, 2, out=out)
    want = [oracle_result(p) for p in parts]
    sums = []
    for mode in (sc.BATCHED, sc.GRAPH, sc.BATCHED):
        per, _ = ctx.reduce(d.tasks, mode)
        for p, g, o in zip(parts, per, want):
            check_result(g, o, p.kid, p.ops, f"kid={p.kid} n={p.n} mode={mode}")
        sums.append([g.sum for g in per])
        shape = ctx.last_launch_shape()
        assert shape["grid"] <= shape["ntiles"] and shape["ntiles"] >= count, shape
    assert sums[0] == sums[1] == sums[2]
    res = torch.zeros(64 * count, dtype=torch.uint8, device="cuda")
    ctx.reduce_noalloc(d.tasks, res)
    torch.cuda.synchronize()
    assert res.view(torch.float64).view(-1, 8)[:, 0].cpu().tolist() == sums[0]
    if out:
        for p, o in zip(parts, d.outs):
            assert not bool(torch.isnan(o).any()), (p.kid, p.n)


def test_caller_tuning_is_taken(ctx):
    # tile tables that the caller sets are the cut, as before
    c = sc.Context(device=0, arena_bytes=64 << 20)
    t = c.get_tuning()
    for m in range(2):
        for k in range(2):
            t.tile[m][k][18] = 1 << 12
    c.set_tuning(t)
    d = DevParts([datagen.make_part(datagen.FMUL, 300_000, i) for i in range(4)])
    c.reduce(d.tasks, sc.BATCHED)
    assert c.last_launch_shape()["ntiles"] == 4 * -(-300_000 // 4096)
    c.destroy()
