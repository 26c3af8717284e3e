"""The solver's kernels with two cells a lane (FP64, n <= 4, from 32768 cells
on), each n and basis a kernel of its own: the V-cycle in the Hermite-type basis
against the same one on vectors that start 8 bytes later (one cell a lane on the
finest level; the arithmetic of a cell does not depend on its lane, so equal
bit for bit), and the iteration with its (r, z) sum, block inverse in FP64 and
FP32, against the same iteration written with the operator, one cycle and dot
products per step."""
import pytest

from paper_2609_04534_amd import tpfdm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cells", [(32, 32, 32), (48, 32, 32)])
def test_hermite_vcycle_on_shifted_vectors(cells):
    import torch
    with tpfdm.Plan.mesh(4, cells, tuple(1.0 / c for c in cells), basis=tpfdm.BASIS_HERMITE) as plan:
        plan.setup_inverse(tpfdm.OP_CELL)
        E = plan.vector_elems
        b = torch.rand(E, dtype=torch.float64, device="cuda",
                       generator=torch.Generator(device="cuda").manual_seed(4)) - 0.5
        bs = torch.empty(E + 1, dtype=torch.float64, device="cuda")[1:]
        bs.copy_(b)
        x = torch.zeros_like(b)
        xs = torch.zeros(E + 1, dtype=torch.float64, device="cuda")[1:]
        with tpfdm.MG(plan) as mg:
            mg.vcycle(b, x)
            mg.vcycle(bs, xs)
            torch.cuda.synchronize()
        assert bool((x == xs).all()) and float(x.abs().max()) > 0.0


@pytest.mark.parametrize("n,basis", [(2, 0), (3, 0), (4, 0), (4, 1)])
@pytest.mark.parametrize("inner", [tpfdm.F64, tpfdm.F32])
def test_iteration_against_its_parts(n, basis, inner):
    import torch
    m = 32   # whole tiles: no padding lanes
    with tpfdm.Plan.mesh(n, (m, m, m), (1.0 / m,) * 3, basis=basis) as plan:
        plan.setup_inverse(tpfdm.OP_CELL)
        g = torch.Generator(device="cuda").manual_seed(n)
        b = torch.rand(plan.vector_elems, dtype=torch.float64, device="cuda", generator=g) - 0.5
        x, z, q = (torch.zeros_like(b) for _ in range(3))
        with tpfdm.MG(plan) as mg, tpfdm.PCG(plan) as solver:
            solver.set_multigrid(mg)
            s = solver.solve(b, x, inner=inner, rtol=1e-4, maxit=50)
            r = b.clone()
            mg.vcycle(r, z)
            p = z.clone()
            rz = float(r @ z)
            its, rel = 0, 1.0
            while rel > 1e-4 and its < 50:
                plan.apply(p, q, tpfdm.OP_SIPG)
                r = r - rz / float(p @ q) * q
                mg.vcycle(r, z)
                rz, old = float(r @ z), rz
                p = z + rz / old * p
                its, rel = its + 1, float(r.norm() / b.norm())
    assert s["iterations"] == its
    # the two differ in the order of sums, and with the FP32 block inverse in the rounding of z
    assert abs(s["relres"] - rel) <= (1e-3 if inner == tpfdm.F32 else 1e-6) * max(rel, 1e-6)
