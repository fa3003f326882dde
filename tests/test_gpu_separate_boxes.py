"""The separate passes of child-region boxes on half the period (k_z, k_inv_y and
k_inv_x of boxes), which NMC_NO_FUSED_PLANES takes from 128 cells on in both
precisions, against the oracle: period 128 and 256, full and partial rows."""
import numpy as np
import pytest
import torch

import oracle
from paper_2301_06763_amd import inputs, nmc

pytestmark = pytest.mark.gpu

TOL = {torch.float64: 1e-12, torch.float32: 1e-5}  # the pointwise bounds of every parity test


@pytest.mark.timeout(180)
@pytest.mark.parametrize("N,L,flags", [(128, 3, 0), (128, 3, nmc.NMC_ONE_STREAM | nmc.NMC_PROLONG_TRILINEAR),
                                       (132, 3, 0), (200, 3, 0)])
def test_separate_boxes_match_oracle(N, L, flags):
    w = inputs.random_levels(N, L, seed=450 + N)
    ref = oracle.solve(w.rho.numpy(), w.h0, trilinear=bool(flags & nmc.NMC_PROLONG_TRILINEAR))
    ctx = nmc.Context()
    try:
        for dtype in (torch.float64, torch.float32):
            print(f"separate boxes N={N} {dtype}", flush=True)
            got = ctx.solve(w.rho.to("cuda", dtype), w.h0, 1.0, flags | nmc.NMC_NO_FUSED_PLANES)
            torch.cuda.synchronize()
            assert np.max(np.abs(got.double().cpu().numpy() - ref) / np.abs(ref)) < TOL[dtype]
    finally:
        ctx.close()


@pytest.mark.timeout(120)
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("N,L,flags", [(32, 3, 0), (64, 2, 0), (20, 3, nmc.NMC_MODIFIED), (16, 3, nmc.NMC_MODIFIED3)])
def test_repeated_calls_read_the_current_input(dtype, N, L, flags):
    """Calls with the same arrays, sizes and stream, each against the oracle of
    what the arrays hold then."""
    w = inputs.random_levels(N, L, seed=480 + N)
    rho = w.rho.to("cuda", dtype)
    out = torch.empty_like(rho)
    ctx = nmc.Context()
    try:
        for k in range(3):
            rho[k % L].mul_(1.0 + k)
            ctx.solve(rho, w.h0, 1.0, flags, out=out)
            torch.cuda.synchronize()
            host = rho.double().cpu().numpy()
            ref = oracle.solve(host, w.h0) if not flags else oracle.solve_modified(
                host, w.h0, scheme="triples" if flags & nmc.NMC_MODIFIED3 else "pairs")
            assert np.max(np.abs(out.double().cpu().numpy() - ref) / np.abs(ref)) < TOL[dtype], k
    finally:
        ctx.close()
