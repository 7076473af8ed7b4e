"""Array reduces where the route or a group's last leaves change, bit for bit
against the oracle's fixed tree: lengths on both sides of the short-array
kernel's 1024 columns, and counts that leave every number of leaves under
eight to a group, as rows and through a pointer table."""
import numpy as np
import pytest
import torch

import oracle
import paper_1505_01120_amd as sc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = sc.Context(device=0, arena_bytes=256 << 20)
    yield c
    c.destroy()


def both(ctx, k, length, comb):
    g = torch.Generator().manual_seed(length * 7919 + k)
    rows = torch.randn(k, length, generator=g)
    want = oracle.tree_reduce_arrays(rows.numpy(), comb).view(np.uint32)
    dev = rows.cuda()
    for call in (lambda out: ctx.reduce_rows(dev, out, comb),
                 lambda out: ctx.reduce_arrays([r for r in dev], out, comb)):
        guard = torch.full((length + 8,), -7.0, device="cuda")
        call(guard[4:4 + length])
        torch.cuda.synchronize()
        assert np.array_equal(guard[4:4 + length].cpu().numpy().view(np.uint32), want)
        assert bool((guard[:4] == -7.0).all()) and bool((guard[4 + length:] == -7.0).all())


@pytest.mark.parametrize("length", [4092, 4093, 4096, 4097, 4100])
@pytest.mark.parametrize("k", [1, 9, 65, 700])
def test_route_edges(ctx, length, k):
    both(ctx, k, length, sc.VADD if k % 2 else sc.VMAX)


@pytest.mark.parametrize("length,groups", [(3, 256), (24, 128), (300, 8), (4096, 1)])
@pytest.mark.parametrize("per", list(range(1, 18)) + [31, 63, 64])
def test_leaves_of_a_group(ctx, length, groups, per):
    # `per` leaves for most groups of a block and one or two fewer for the last
    both(ctx, max(1, min(groups, 4096 // per) * per - per % 3), length,
         sc.VMAX if per % 2 else sc.VADD)
