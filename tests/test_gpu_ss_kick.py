"""The split-step kick exp(i sigma |A|^2 dz) where a thread's eight points
straddle the bound of its polynomial (|phi| <= 1/64 at all of them) and where
none is below it, against the oracle's Eq. 4, in the one-workgroup and the
four-step path.  The tolerances are the suite's; the steps are few, so the
stored field's rounding (2^-24 a step in FP32) stays far below 1e-5."""
import numpy as np
import pytest

import oracle as O
from tests.gpu_util import TOL_F32, TOL_F64, rel_l2, say, to_dev, to_host
from workloads import Grid, dm_map, wdm_field

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,prec", [(512, 1), (4096, 0), (4096, 1), (8192, 1), (65536, 0)])
@pytest.mark.parametrize("peak", [1.0 / 64, 2.0])
def test_kick_beyond_the_polynomial(n, prec, peak):
    import paper_1101_0086_amd as P
    grid = Grid(n, 10.0 / 256)
    a = wdm_field(grid, n // 256, 1, "qpsk", np.random.default_rng(n + prec))
    dz = 1.0 / 320
    # the largest phase of the first kick: on the bound (most points below it), or far above
    sigma = peak / (dz * float(np.max(np.abs(a)) ** 2))
    dmm = dm_map(beta3=0.0, sigma=sigma)
    say("kick", n, prec, peak)
    plan = P.SSPlan(n, grid.dt, dmm, dz, prec)
    x = to_dev(a, prec)
    plan.propagate(x, 0.0, 8 * dz)
    ref = O.ss_propagate(a, grid.dt, dmm, dz, 0.0, 8 * dz)
    assert rel_l2(to_host(x), ref) < (TOL_F32 if prec == 0 else TOL_F64)
    plan.close()
