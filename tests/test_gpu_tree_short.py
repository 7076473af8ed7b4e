"""Array-valued ReduceCL over short arrays (thread groups combined in LDS) and
over lengths that are no multiple of 4 (a last quad that overlaps the one
before), bit for bit against the oracle's fixed tree."""
import numpy as np
import pytest
import torch

import oracle
import paper_1505_01120_amd as sc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = sc.Context(device=0, arena_bytes=1 << 30)
    yield c
    c.destroy()


def same(got, host, comb):
    want = oracle.tree_reduce_arrays(host, comb)
    return np.array_equal(got.cpu().numpy().view(np.uint32), want.view(np.uint32))


# lengths at the edges of a quad, of a block's columns (512 quads) and of its
# powers of two; counts at the edges of a thread's 8-leaf groups, of one
# block and of several passes
@pytest.mark.parametrize("length", [1, 2, 3, 4, 5, 7, 24, 27, 129, 1021, 1028, 2045, 2048, 2049])
@pytest.mark.parametrize("k", [1, 2, 9, 65, 513, 4100, 33000])
def test_rows(ctx, length, k):
    if k * length > 1 << 23:
        k = (1 << 23) // length
    g = torch.Generator().manual_seed(length * 131 + k)
    for pad, comb in ((0, sc.VADD), (1, sc.VMAX)):
        rows = torch.randn(k, length + pad, generator=g)
        dev = rows.cuda()[:, :length]
        guard = torch.full((length + 8,), -7.0, device="cuda")
        ctx.reduce_rows(dev, guard[4:4 + length], comb)
        torch.cuda.synchronize()
        assert same(guard[4:4 + length], np.ascontiguousarray(rows[:, :length].numpy()), comb)
        assert bool((guard[:4] == -7.0).all()) and bool((guard[4 + length:] == -7.0).all())


# pointer tables, out over one of the inputs: the short kernel, the column
# kernel and the wide one (2 and 4 columns, 256 and 512 threads)
@pytest.mark.parametrize("k,length", [(5, 6), (700, 31), (33, 2050), (48, 100003),
                                      (3, (1 << 20) + 1), (9, (1 << 21) + 3),
                                      (3, 4 * (2048 * 512 + 100) + 2)])
def test_ragged_arrays_in_place(ctx, k, length):
    g = torch.Generator(device="cuda").manual_seed(k)
    flat = torch.randn(k, length + 1, device="cuda", generator=g)
    rows = [r[1:] for r in flat]
    at = np.unique(np.r_[0:min(length, 3000), max(0, length - 3000):length])
    host = flat[:, 1:].cpu().numpy()[:, at]
    ctx.reduce_arrays(rows, rows[k // 2], sc.VADD)
    torch.cuda.synchronize()
    got = rows[k // 2][torch.from_numpy(at).cuda()]
    assert same(got, np.ascontiguousarray(host), sc.VADD)
    assert bool((flat[:, 0] == torch.randn(k, length + 1, device="cuda",
                 generator=torch.Generator(device="cuda").manual_seed(k))[:, 0]).all())
