"""nmc_solve captured into a HIP graph: its workspace and tables are its own, so
replays between other solves equal the solve alone, on new inputs too."""
import pytest
import torch

from paper_2301_06763_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.timeout(120)
@pytest.mark.parametrize("N,L,dtype", [(16, 3, torch.float64), (48, 2, torch.float32), (128, 2, torch.float64)])
def test_replays_between_other_solves(N, L, dtype):
    from paper_2301_06763_amd import nmc
    c = nmc.Context()
    try:
        s = torch.cuda.Stream()
        rho = inputs.random_levels(N, L, seed=310 + N).rho.to("cuda", dtype)
        others = [inputs.random_levels(n, 3, seed=320 + n).rho.to("cuda", dtype) for n in (N, 2 * N if N < 64 else 64, 20)]
        out = torch.empty_like(rho)
        torch.cuda.synchronize()
        # the tables, and a cached block for the captured call: nothing is allocated in it
        big = inputs.random_levels(N, L + 1, seed=330).rho.to("cuda", dtype)
        torch.cuda.synchronize()
        c.solve(rho, 0.1, out=out, stream=s)
        c.solve(big, 0.1, out=torch.empty_like(big), stream=s)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s, capture_error_mode="relaxed"):
            c.solve(rho, 0.1, out=out, stream=s)
        alone = [c.solve(o, 0.1) for o in others]
        torch.cuda.synchronize()
        for k in range(4):
            rho.mul_(1.0 + 0.25 * k)
            torch.cuda.synchronize()
            with torch.cuda.stream(s):
                g.replay()
            got = [c.solve(o, 0.1) for o in others]  # on the default stream, beside the replay
            torch.cuda.synchronize()
            assert torch.equal(out, c.solve(rho, 0.1)), k
            for a, b in zip(got, alone):
                assert torch.equal(a, b), k
        del g
    finally:
        torch.cuda.synchronize()
        c.close()
