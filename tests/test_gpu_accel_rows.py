"""nmc_acceleration with vector rows (N >= 20, 16-byte aligned arrays) against
the one-cell kernel that the same call takes for an array off that alignment:
the same values, at the smallest sizes, rows that end inside a workgroup and
odd child-region offsets."""
import pytest
import torch

from paper_2301_06763_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.timeout(120)
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("N,L", [(16, 2), (20, 1), (20, 3), (24, 2), (28, 3), (64, 2), (96, 2), (100, 3)])
def test_rows_equal_cells(dtype, N, L):
    from paper_2301_06763_amd import nmc
    ctx = nmc.Context()
    try:
        phi = inputs.random_levels(N, L, seed=40 + N).rho.to("cuda", dtype)
        off = torch.empty(phi.numel() + 1, dtype=dtype, device="cuda")[1:].view_as(phi)
        off.copy_(phi)
        assert phi.data_ptr() % 16 == 0 and off.data_ptr() % 16 != 0
        a, b = ctx.acceleration(phi, 1 / N), ctx.acceleration(off, 1 / N)
        torch.cuda.synchronize()
        assert torch.equal(a, b)
    finally:
        ctx.close()


# where the rule takes vector rows at the smallest N of each type, and sizes on
# both sides of its line (L N^3 from 25 000 in FP64, 130 000 in FP32)
@pytest.mark.timeout(120)
@pytest.mark.parametrize("dtype,N,L", [(torch.float64, 20, 3), (torch.float64, 20, 4), (torch.float64, 28, 2),
                                       (torch.float32, 24, 10), (torch.float32, 28, 6), (torch.float32, 40, 2),
                                       (torch.float32, 44, 2), (torch.float32, 52, 1)])
def test_rows_from_enough_cells(dtype, N, L):
    test_rows_equal_cells(dtype, N, L)
