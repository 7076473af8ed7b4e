"""Calls made while the serving executor is resident run beside it: they end
long before it would leave, and it is still there afterwards."""
import time

import pytest
import torch

import paper_1505_01120_amd as sc

pytestmark = pytest.mark.gpu

IDLE_MS = 2000


@pytest.fixture(scope="module")
def ctx():
    c = sc.Context(device=0, arena_bytes=512 << 20, idle_exit_ms=IDLE_MS)
    yield c
    c.destroy()


def calls(ctx):
    x = torch.randn(1 << 22, device="cuda")
    out = torch.empty(1 << 22, device="cuda")
    short = x[:24 * 100000].view(-1, 24)
    rows = x.view(-1, 4096)
    yield "rows of 24", lambda: ctx.reduce_rows(short, out[:24], sc.VADD)
    yield "rows of 4096", lambda: ctx.reduce_rows(rows, out[:4096], sc.VMAX)
    yield "arrays", lambda: ctx.reduce_arrays([r for r in rows[:300]], out[:4096], sc.VADD)
    task = sc.task(sc.POLY, 1 << 22, x, out=out, coef=(1.0, 2.0))
    yield "map", lambda: ctx.map([task])
    yield "reduce", lambda: ctx.reduce([task], sc.BATCHED)
    yield "Monte-Carlo", lambda: ctx.reduce([sc.task(sc.MC_PI, 1 << 22)], sc.BATCHED)


def check(ctx, named):
    named = list(named)
    x = torch.ones(1000, device="cuda")
    served = sc.task(sc.POLY, 1000, x, coef=(0.0, 1.0))

    def serve():
        ticket = ctx.submit(served)
        end = time.monotonic() + 10
        while time.monotonic() < end:
            r = ctx.poll(ticket)
            if r is not None:
                return r.sum
        raise AssertionError("served task not done")

    for _, call in named:  # plans, code objects and pinned buffers
        call()
    torch.cuda.synchronize()
    for name, call in named:
        assert serve() == 1000.0
        launches = ctx.serve_stats()["executor_launches"]
        t0 = time.monotonic()
        call()
        torch.cuda.current_stream().synchronize()
        took = time.monotonic() - t0
        assert took < IDLE_MS / 4000, f"{name} took {took * 1e3:.0f} ms"
        assert serve() == 1000.0
        assert ctx.serve_stats()["executor_launches"] == launches, f"{name}: executor had left"


def test_calls_beside_serving(ctx):
    check(ctx, calls(ctx))


@pytest.mark.parametrize("nbytes", [1 << 12, 1 << 20, 1 << 26])
def test_wordcount_beside_serving(ctx, nbytes):
    g = torch.Generator(device="cuda").manual_seed(nbytes)
    text = torch.randint(97, 123, (nbytes,), device="cuda", generator=g).to(torch.uint8)
    text[::4] = 32
    cap = 1 << 15
    keys, counts, distinct, _ = ctx.wordcount(text, cap)
    found = keys[:distinct].clone()
    offsets = torch.empty_like(found)
    check(ctx, [("word count", lambda: ctx.wordcount(text, cap, keys, counts)),
                ("locate", lambda: ctx.wordcount_locate(text, found, offsets=offsets))])
