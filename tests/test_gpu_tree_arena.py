"""Array reduces in the smallest arena: shapes whose rows take little scratch,
and ones that only the plan with the fewest rows fits, bit for bit as in a
large arena."""
import pytest
import torch

import paper_1505_01120_amd as sc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,length", [(65536, 4096), (1 << 17, 3000), (4096, 4097), (4097, 4099),
                                      (300000, 255), (128, (1 << 22) + 1), (5000, 100003)])
@pytest.mark.parametrize("comb", [sc.VADD, sc.VMAX])
def test_small_arena(k, length, comb):
    g = torch.Generator(device="cuda").manual_seed(length)
    rows = torch.randn(k, length, device="cuda", generator=g)
    got, want = (torch.empty(length, device="cuda") for _ in range(2))
    with sc.Context(device=0, arena_bytes=16 << 20) as small:
        small.reduce_rows(rows, got, comb)
        torch.cuda.synchronize()
    with sc.Context(device=0, arena_bytes=1 << 30) as large:
        large.reduce_rows(rows, want, comb)
        torch.cuda.synchronize()
    assert torch.equal(got.view(torch.int32), want.view(torch.int32))
