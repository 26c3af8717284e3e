"""MG-PCG solves with every split of check_every into captured graphs (a graph
holds the largest divisor up to 4 of check_every; a chunk of the non-blocking
solve launches several): the iterations run on the device, so iterate, count
and residual are equal bit for bit, also after the chunk size changes on one
solver, and maxit stops inside a graph."""
import pytest

from paper_2609_04534_amd import tpfdm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m", [(3, 8), (5, 4)])
def test_chunk_sizes_agree(n, m):
    import torch
    with tpfdm.Plan.mesh(n, (m, m, m), (1.0 / m,) * 3) as plan:
        plan.setup_inverse(tpfdm.OP_CELL)
        b = torch.rand(plan.vector_elems, dtype=torch.float64, device="cuda",
                       generator=torch.Generator(device="cuda").manual_seed(5)) - 0.5
        with tpfdm.MG(plan) as mg, tpfdm.PCG(plan) as cg:
            cg.set_multigrid(mg)
            ref = None
            for k in (16, 1, 3, 5, 6, 8):
                x = torch.zeros_like(b)
                out = cg.solve(b, x, check_every=k, rtol=1e-9)
                y = torch.zeros_like(b)
                cg.begin(b, y, check_every=k, rtol=1e-9)
                poll = None
                while poll is None:
                    poll = cg.poll()
                torch.cuda.synchronize()
                if ref is None:
                    ref = (out, x)
                assert out["converged"] and out == ref[0] and poll == ref[0]
                assert bool((x == ref[1]).all()) and bool((y == ref[1]).all())
            for maxit in (0, 1, 3):
                x = torch.zeros_like(b)
                out = cg.solve(b, x, maxit=maxit, rtol=1e-9, raise_on_failure=False)
                assert out["iterations"] == maxit and not out["converged"]
