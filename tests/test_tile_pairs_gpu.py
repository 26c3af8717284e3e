"""The coupled operator with two cells a lane (FP64, n <= 4, an even cell
count in z, 32768 cells or more, 16-byte aligned vectors) against the same
call on vectors that start 8 bytes later, which runs one cell a lane: the
arithmetic of a cell does not depend on the lane it runs in, so every value
is equal bit for bit.  Boxes at the smallest count, with a ragged last
workgroup (counts not a multiple of 128, workgroup counts not a multiple of
8), pairs at z faces (two cells in z), one-cell-thick directions; the outputs
start as NaN, and sampled cells are checked against the oracle's row blocks
(FP64 rounding of at most 8 n^4 terms: 1e-12 of max |A||u|)."""
import numpy as np
import pytest

from oracle import sipg
from paper_2609_04534_amd import tpfdm

from .gpu_util import from_blocked

pytestmark = pytest.mark.gpu

BOXES = [(32, 32, 32), (33, 31, 34), (128, 129, 2), (1, 250, 132), (400, 1, 90)]


@pytest.mark.parametrize("n,basis", [(2, 0), (3, 0), (4, 0), (4, 1)])
@pytest.mark.parametrize("cells", BOXES)
def test_two_cells_a_lane_equal_one(n, basis, cells):
    import torch
    ncell = int(np.prod(cells))
    h = (0.05, 0.03, 0.04)
    plan = tpfdm.Plan.mesh(n, cells, h, basis=basis)
    with plan:
        E = plan.vector_elems
        u = torch.rand(E + 2, dtype=torch.float64, device="cuda",
                       generator=torch.Generator(device="cuda").manual_seed(n)) - 0.5
        ua, ub = u[:E].clone(), torch.empty(E + 1, dtype=torch.float64, device="cuda")[1:]
        ub.copy_(ua)
        assert ua.data_ptr() % 16 == 0 and ub.data_ptr() % 16 == 8
        va = torch.full_like(ua, float("nan"))
        vb = torch.full((E + 1,), float("nan"), dtype=torch.float64, device="cuda")[1:]
        plan.apply(ua, va, tpfdm.OP_SIPG)
        plan.apply(ub, vb, tpfdm.OP_SIPG)
        ga, gb = from_blocked(plan, va, tpfdm.F64), from_blocked(plan, vb.clone(), tpfdm.F64)
        assert np.isfinite(ga).all()
        assert np.array_equal(ga, gb)
        if basis == 0:
            uc = from_blocked(plan, ua, tpfdm.F64).reshape(ncell, -1)
            rng = np.random.default_rng(n)
            cs = [0, ncell - 1, 63, 64, 127, 128] + rng.choice(ncell, 10, replace=False).tolist()
            for c in cs:
                ref = scale = 0.0
                for nb, blk in sipg.cell_row_blocks(n - 1, cells, h, c):
                    ref = ref + blk @ uc[nb]
                    scale = scale + np.abs(blk) @ np.abs(uc[nb])
                assert np.max(np.abs(ga.reshape(ncell, -1)[c] - ref)) <= 1e-12 * np.max(scale)


@pytest.mark.parametrize("n", [2, 3, 4])
@pytest.mark.parametrize("cells", [(8, 8, 8), (32, 32, 32)])
def test_vcycle_on_shifted_vectors(n, cells):
    """One V-cycle on vectors that start 8 bytes later (one cell a lane on the
    finest level, right-hand side pairs at 8-byte alignment in the restriction)
    equals the aligned one bit for bit."""
    import torch
    with tpfdm.Plan.mesh(n, cells, tuple(1.0 / c for c in cells)) as plan:
        plan.setup_inverse(tpfdm.OP_CELL)
        E = plan.vector_elems
        b = torch.rand(E, dtype=torch.float64, device="cuda",
                       generator=torch.Generator(device="cuda").manual_seed(n)) - 0.5
        bs = torch.empty(E + 1, dtype=torch.float64, device="cuda")[1:]
        bs.copy_(b)
        x = torch.zeros_like(b)
        xs = torch.zeros(E + 1, dtype=torch.float64, device="cuda")[1:]
        with tpfdm.MG(plan) as mg:
            mg.vcycle(b, x)
            mg.vcycle(bs, xs)
            torch.cuda.synchronize()
        assert bool((x == xs).all()) and float(x.abs().max()) > 0.0
