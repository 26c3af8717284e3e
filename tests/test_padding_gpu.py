"""Padding lanes of a ragged last tile are the caller's: V-cycles and solves
leave them as they were (with FP32 level storage a V-cycle, and every solve,
used to copy their whole inner vector, whose padding nothing writes)."""
import pytest

from paper_2609_04534_amd import tpfdm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,cells", [(2, (1, 1, 1)), (3, (3, 5, 2)), (3, (4, 6, 10)), (4, (2, 3, 1)), (5, (2, 2, 2))])
def test_padding_lanes_are_not_written(n, cells):
    import torch
    with tpfdm.Plan.mesh(n, cells, tuple(1.0 / c for c in cells)) as plan:
        plan.setup_inverse(tpfdm.OP_CELL)
        cell = torch.zeros(plan.vector_elems, dtype=torch.float64, device="cuda")
        plan.pack(torch.ones(plan.ndof, dtype=torch.float64, device="cuda"), cell)
        pad = cell == 0
        assert int(pad.sum()) == plan.vector_elems - plan.ndof
        b = torch.rand(plan.vector_elems, dtype=torch.float64, device="cuda",
                       generator=torch.Generator(device="cuda").manual_seed(n)) - 0.5
        zero = torch.zeros_like(b)
        for storage in (tpfdm.F64, tpfdm.F32):
            with tpfdm.MG(plan, storage=storage) as mg, tpfdm.PCG(plan) as cg:
                def check(call):
                    x = torch.where(pad, torch.full_like(b, 7.0), zero)
                    call(x)
                    torch.cuda.synchronize()
                    assert bool((x[pad] == 7.0).all()) and bool(torch.isfinite(x).all())
                    assert float(x[~pad].abs().max()) > 0.0
                    return x

                def begun(x):
                    cg.begin(b, x)
                    while cg.poll() is None:
                        pass

                check(lambda x: mg.vcycle(b, x))
                for m in (None, mg):
                    cg.set_multigrid(m)
                    x = check(lambda x: cg.solve(b, x))
                    y = check(begun)
                    assert bool((x == y).all())
