"""Residual and restriction of the multigrid levels for n >= 5 in one launch:
one V-cycle against the oracle's on boxes whose coarse cells are no multiple
of eight, level vectors in FP64 and FP32."""
import numpy as np
import pytest

from oracle import mg
from paper_2609_04534_amd import tpfdm
from tests.gpu_util import from_blocked, to_blocked

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p,cells", [(4, (10, 6, 2)), (5, (10, 2, 2)), (6, (6, 2, 2)), (7, (2, 6, 2))])
@pytest.mark.parametrize("storage,tol", [(tpfdm.F64, 1e-11), (tpfdm.F32, 2e-5)])
def test_vcycle_with_ragged_coarse_level(p, cells, storage, tol):
    import torch
    h = tuple(1.0 / c for c in cells)
    H = mg.Hierarchy(p, cells, h=h)
    b = np.random.default_rng(sum(cells) + p).uniform(-1, 1, H.A[0].shape[0])
    xo = H.vcycle(b)
    with tpfdm.Plan.mesh(p + 1, cells, h) as plan:
        plan.setup_inverse(tpfdm.OP_CELL)
        with tpfdm.MG(plan, storage=storage) as V:
            bb = to_blocked(plan, b, tpfdm.F64)
            bx = torch.full_like(bb, float("nan"))
            V.vcycle(bb, bx)
            x = from_blocked(plan, bx, tpfdm.F64)
    assert np.all(np.isfinite(x))
    assert np.abs(x - xo).max() <= tol * np.abs(xo).max()
