"""The coupled operator with one cell per wave (n = 5..8) on a box whose
x-planes are visited in groups with a narrower last group and a plain-order
tail (221 cells per plane, groups of 192): the output starts as NaN, sampled
cells are checked against the oracle's row blocks (FP64 1e-12, FP32 2e-6 of
max |A||u|), and at n = 8 in FP64 the 16-byte neighbour loads give, bit for
bit, the result of the scalar ones (the same call on vectors 8 bytes later:
one cell's arithmetic does not depend on how its values are loaded), also on
one-cell-thick boxes, where both faces of an axis lie on the boundary."""
import numpy as np
import pytest

from oracle import sipg
from paper_2609_04534_amd import tpfdm

from .gpu_util import from_blocked

pytestmark = pytest.mark.gpu

TOL = {tpfdm.F64: 1e-12, tpfdm.F32: 2e-6}


def _apply(plan, E, dt, shift):
    import torch
    t = torch.float64 if dt == tpfdm.F64 else torch.float32
    u = torch.rand(E, dtype=t, device="cuda", generator=torch.Generator(device="cuda").manual_seed(3)) - 0.5
    us, vs = (torch.full((E + shift,), float("nan"), dtype=t, device="cuda")[shift:] for _ in range(2))
    us.copy_(u)
    plan.apply(us, vs, tpfdm.OP_SIPG)
    return u, vs.clone()


@pytest.mark.parametrize("n", [5, 6, 7, 8])
@pytest.mark.parametrize("dt", [tpfdm.F64, tpfdm.F32])
def test_grouped_cells(n, dt):
    cells, h = (17, 13, 17), (0.05, 0.03, 0.04)
    ncell = int(np.prod(cells))
    with tpfdm.Plan.mesh(n, cells, h) as plan:
        u, v = _apply(plan, plan.vector_elems, dt, 0)
        uc = from_blocked(plan, u, dt).reshape(ncell, -1).astype(np.float64)
        got = from_blocked(plan, v, dt).reshape(ncell, -1).astype(np.float64)
        assert np.isfinite(got).all()
        rng = np.random.default_rng(n)
        for c in [0, ncell - 1, 191, 192, 220, 221] + rng.choice(ncell, 6, replace=False).tolist():
            ref = scale = 0.0
            for nb, blk in sipg.cell_row_blocks(n - 1, cells, h, c):
                ref = ref + blk @ uc[nb]
                scale = scale + np.abs(blk) @ np.abs(uc[nb])
            assert np.max(np.abs(got[c] - ref)) <= TOL[dt] * np.max(scale)


@pytest.mark.parametrize("basis", [0, 1])
@pytest.mark.parametrize("cells", [(17, 13, 17), (1, 5, 1), (5, 1, 3), (1, 1, 4)])
def test_vector_loads_equal_scalar_loads(basis, cells):
    with tpfdm.Plan.mesh(8, cells, (0.05, 0.03, 0.04), basis=basis) as plan:
        E = plan.vector_elems
        _, a = _apply(plan, E, tpfdm.F64, 0)
        _, b = _apply(plan, E, tpfdm.F64, 1)
        assert bool(a.isfinite().all()) and bool((a == b).all())
