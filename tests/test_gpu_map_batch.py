"""MapCL over many tasks in one launch, bit-exact against the oracle: sizes at
the edges of a block's tile (4096 elements), tasks without elements among
them, more tasks than one wave's search reads, and tasks that feed each other.
"""
import numpy as np
import pytest
import torch

import datagen
import oracle
import paper_1505_01120_amd as sc
from gpu_helpers import dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = sc.Context(device=0, arena_bytes=256 << 20)
    yield c
    c.destroy()


def bits(a):
    return (a.cpu().numpy() if hasattr(a, "cpu") else a).view(np.uint32)


def run(ctx, sizes, xoff, ooff):
    tasks, want, outs = [], [], []
    for i, n in enumerate(sizes):
        p = datagen.make_part(datagen.POLY if i % 2 else datagen.FMUL, n, i)
        x, y = dev(p.x, xoff), dev(p.y, (xoff + i) % 4) if p.y is not None else None
        buf = torch.full((n + 8,), float("nan"), device="cuda")
        tasks.append(sc.task(p.kid, n, x, y, buf[ooff:ooff + n], coef=p.coef, c=p.c))
        want.append(oracle.poly_map(p.x, p.coef) if p.kid == datagen.POLY
                    else oracle.fmul_map(p.x, p.y))
        outs.append((x, y, buf))
    ctx.map(tasks)
    ctx.map(tasks)  # the cached plan
    torch.cuda.synchronize()
    for i, (n, w, (_, _, buf)) in enumerate(zip(sizes, want, outs)):
        assert np.array_equal(bits(buf[ooff:ooff + n]), bits(w)), (i, n)
        assert torch.isnan(buf[:ooff]).all() and torch.isnan(buf[ooff + n:]).all(), (i, n)


@pytest.mark.parametrize("xoff,ooff", [(0, 0), (1, 0), (3, 2)])
def test_tile_edges(ctx, xoff, ooff):
    run(ctx, [1, 3, 4, 5, 0, 1023, 1024, 1025, 4095, 4096, 4097, 4099, 4100, 0, 0, 8191, 8192,
              8193, 8195, 12288, 65537, 0], xoff, ooff)


@pytest.mark.parametrize("count", [63, 64, 65, 129, 4097])
def test_many_tasks(ctx, count):
    rng = np.random.RandomState(count)
    run(ctx, [int(v) for v in rng.choice([0, 1, 7, 64, 4096, 5000, 9001], count)], 0, 1)


def test_tasks_that_feed_each_other_run_in_order(ctx):
    n = 200_003
    x = datagen.fill(n, 3, 0, 1, datagen.U_PM1)
    a, b, c = dev(x), dev(np.zeros(n, np.float32)), dev(np.zeros(n, np.float32), 1)
    coef = (0.5, 0.25, -0.75)
    tasks = [sc.task(sc.POLY, n, a, None, b, coef=coef),      # b = p(a)
             sc.task(sc.FMUL, n, b, a, c, c=0.1),             # c = b a + 0.1 b
             sc.task(sc.POLY, n, c, None, c, coef=coef)]      # c = p(c), in place
    ctx.map(tasks)
    torch.cuda.synchronize()
    pb = oracle.poly_map(x, coef)
    pc = oracle.poly_map(oracle.fmul_map(pb, x), coef)
    assert np.array_equal(bits(b), bits(pb)) and np.array_equal(bits(c), bits(pc))
