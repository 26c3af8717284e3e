"""(r, z) of the multigrid-preconditioned iteration, which the cycle's last
update sums: the solver's iterations and final residual against the same
iteration written with the operator, one cycle and dot products per step.
Sizes: finest level below, at and above one workgroup, one and two cells a
lane, one cell a wave, and single-level hierarchies."""
import pytest

from paper_2609_04534_amd import tpfdm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,cells", [(2, (1, 1, 1)), (3, (4, 4, 4)), (4, (8, 8, 8)), (4, (6, 10, 4)), (2, (32, 32, 32)),
                                     (5, (6, 6, 6)), (8, (4, 2, 6)), (8, (3, 3, 3))])
@pytest.mark.parametrize("storage", [tpfdm.F64, tpfdm.F32])
def test_iteration_against_its_parts(n, cells, storage):
    import torch
    with tpfdm.Plan.mesh(n, cells, tuple(1.0 / c for c in cells)) as plan:
        plan.setup_inverse(tpfdm.OP_CELL)
        # the mesh's unknowns: no padding of the vectors may enter the sums
        b = torch.ones(plan.vector_elems, dtype=torch.float64, device="cuda")
        used = torch.zeros_like(b)
        plan.apply(b, used, tpfdm.OP_CELL)
        used = (used != 0).to(b.dtype)
        g = torch.Generator(device="cuda").manual_seed(n)
        b = (torch.rand(plan.vector_elems, dtype=torch.float64, device="cuda", generator=g) - 0.5) * used
        xs, z, q = (torch.zeros_like(b) for _ in range(3))
        with tpfdm.MG(plan, storage=storage) as mg, tpfdm.PCG(plan) as solver:
            solver.set_multigrid(mg)
            s = solver.solve(b, xs, rtol=1e-4, maxit=50)
            r = b.clone()
            mg.vcycle(r, z)
            p = z * used
            rz = float(r @ p)
            its, rel = 0, 1.0
            while rel > 1e-4 and its < 50:
                plan.apply(p, q, tpfdm.OP_SIPG)
                r = r - rz / float(p @ (q * used)) * q * used
                mg.vcycle(r, z)
                z = z * used
                rz, old = float(r @ z), rz
                p = z + rz / old * p
                its, rel = its + 1, float(r.norm() / b.norm())
    assert s["iterations"] == its
    # the two differ in the order of sums, and in FP32 also in the rounding of z
    assert abs(s["relres"] - rel) <= (1e-3 if storage == tpfdm.F32 else 1e-6) * max(rel, 1e-6)
