"""nmc_solve_noalloc on the tables that another call left: a solve of another size
of the same period, another method, or the other choice of passes."""
import numpy as np
import pytest
import torch

import oracle
from paper_2301_06763_amd import inputs, nmc

pytestmark = pytest.mark.gpu

TOL = {torch.float64: 1e-12, torch.float32: 1e-5}  # the pointwise bounds of every parity test


@pytest.mark.timeout(120)
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("left,asked", [
    ((64, 0), (48, 0)), ((36, nmc.NMC_NO_FUSED_PLANES), (60, 0)), ((48, 0), (64, nmc.NMC_NO_FUSED_PLANES)),
    ((36, nmc.NMC_MODIFIED), (36, nmc.NMC_MODIFIED | nmc.NMC_NO_FUSED_PLANES)),
    ((40, nmc.NMC_MODIFIED), (36, 0)), ((32, nmc.NMC_MODIFIED), (64, 0)),
])
def test_tables_another_call_left(dtype, left, asked):
    c = nmc.Context()
    try:
        c.solve(inputs.random_levels(left[0], 2, seed=1).rho.to("cuda", dtype), 0.1, flags=left[1])
        N, flags = asked
        w = inputs.random_levels(N, 2, seed=840 + N)
        got = c.solve_noalloc(w.rho.to("cuda", dtype), w.h0, flags=flags)
        torch.cuda.synchronize()
        mod = flags & nmc.NMC_MODIFIED
        ref = oracle.solve_modified(w.rho.numpy(), w.h0, scheme="pairs") if mod else oracle.solve(w.rho.numpy(), w.h0)
        assert np.max(np.abs(got.double().cpu().numpy() - ref) / np.abs(ref)) < TOL[dtype]
    finally:
        c.close()
