"""Kernel ids that name no kernel are refused by every call, on a context that
cuts small batches by estimated time."""
import pytest
import torch

import paper_1505_01120_amd as sc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kid", [0, 4, 10, 100, 0xFFFFFFFF])
def test_unknown_kernel(kid):
    x = torch.zeros(5000, dtype=torch.float32, device="cuda")
    res = torch.zeros(2 * 64, dtype=torch.uint8, device="cuda")
    good = sc.task(sc.POLY, 5000, x, coef=(1.0, 2.0))
    bad = sc.Task(kernel_id=kid, reduce_ops=sc.SUM, n=5000, in0=x.data_ptr(), in1=x.data_ptr())
    with sc.Context(device=0, arena_bytes=64 << 20) as ctx:
        for tasks in ([bad], [good, bad]):
            for mode in (sc.PER_LAUNCH, sc.BATCHED, sc.GRAPH):
                for call in (lambda: ctx.reduce(tasks, mode),
                             lambda: ctx.reduce_async(tasks, mode, res)):
                    with pytest.raises(sc.SparkclError) as e:
                        call()
                    assert e.value.code == sc.ENOKERNEL, (kid, mode)
            for call in (lambda: ctx.reduce_noalloc(tasks, res),
                         lambda: ctx.reduce_chain(tasks, [sc.stage((0.5, 2.0))])):
                with pytest.raises(sc.SparkclError) as e:
                    call()
                assert e.value.code == sc.ENOKERNEL, kid
        per, _ = ctx.reduce([good], sc.BATCHED)
        assert per[0].sum == 5000.0
