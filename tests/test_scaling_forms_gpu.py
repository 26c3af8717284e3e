"""Product and inverse of one-block tiles (n = 6, 7, 8) on 16-byte aligned
vectors, on vectors one element later and in the layout B = 64: at n = 8 the
last two compute a block's scalings in every lane, the first in three lanes,
and the loads differ; the arithmetic does not, so the results are equal bit
for bit."""
import numpy as np
import pytest

from paper_2609_04534_amd import tpfdm

from .gpu_util import canon, from_blocked, to_blocked

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [6, 7, 8])
@pytest.mark.parametrize("dt", [tpfdm.F64, tpfdm.F32])
@pytest.mark.parametrize("nb", [1, 37, 5000])
def test_scalings_in_three_lanes_or_in_all(n, dt, nb):
    import torch
    rng = np.random.default_rng(n)
    h, u = rng.uniform(0.5, 4.0, (nb, 3)), rng.uniform(-1, 1, (nb, n ** 3))
    got = []
    for B, shift in ((1, 0), (1, 1), (64, 0)):
        with tpfdm.Plan([tpfdm.GroupSpec(n, B, h)]) as plan:
            plan.setup_inverse(tpfdm.OP_CELL)
            a = to_blocked(plan, canon([u]), dt)
            bu = torch.zeros(a.numel() + shift, dtype=a.dtype, device="cuda")[shift:]
            bu.copy_(a)
            out = []
            for call in (lambda v: plan.apply(bu, v, tpfdm.OP_CELL), lambda v: plan.apply_inverse(bu, v)):
                v = torch.full((a.numel() + shift,), float("nan"), dtype=a.dtype, device="cuda")[shift:]
                call(v)
                out.append(from_blocked(plan, v.clone(), dt))
            got.append(np.stack(out))
    assert np.isfinite(got[0]).all()
    assert np.array_equal(got[0], got[1]) and np.array_equal(got[0], got[2])
