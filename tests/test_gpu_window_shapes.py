"""Long steps on windows above 4096 modes where their row pass takes each of
its roles: a single evaluation (M = 1, one sweep: the first evaluation is the
last), one node with several sweeps, several nodes with one sweep; rows of 128
to 2048 points, columns of 64 to 1024.  Against the oracle's full-window march;
tolerances of the suite."""
import numpy as np
import pytest

import oracle as O
from tests.gpu_util import TOL_F32, TOL_F64, rel_l2, say, to_dev, to_host
from workloads import Grid, dm_map
from workloads.wdm import _fast_wdm_field

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("lg,M,nit", [(13, 1, 1), (14, 1, 3), (15, 3, 1), (16, 2, 2), (18, 1, 2), (21, 1, 1)])
def test_window_evaluation_counts(lg, M, nit, prec):
    import paper_1101_0086_amd as P
    n, dt = 1 << lg, 10.0 / 1024
    a = _fast_wdm_field(Grid(n, dt), n // 1024, 8, "qpsk", np.random.default_rng(lg))
    dmm = dm_map(beta3=0.1)
    L = 2.5e-4
    steps = 1 if lg > 16 else 3
    z0 = 0.5 - (steps // 2) * L                 # several steps cross the span change
    say("window", lg, M, nit, prec)
    plan = P.MPAPlan(n, dt, dmm, L, M, nit, 0, 0, prec)
    x = to_dev(a, prec)
    plan.propagate(x, z0, z0 + steps * L)
    got = to_host(x)
    plan.close()
    ref = O.mpa_propagate(a, dt, dmm, L, M, nit, z0, z0 + steps * L)
    assert rel_l2(got, ref) < (TOL_F32 if prec == 0 else TOL_F64)
