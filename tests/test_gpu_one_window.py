"""One full window of at most 4096 modes marches in place; on the node-parallel
kernels each long step's last launch also starts the next one.  A march equals
its steps one by one (bitwise), in odd and even numbers, across a span change
and an amplifier, and the oracle within the suite's tolerances."""
import numpy as np
import pytest

import oracle as O
from tests.gpu_util import TOL_F32, TOL_F64, rel_l2, say, to_dev, to_host
from workloads import Grid, dm_map, wdm_field

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n,M,nit,sched", [(512, 1, 2, 0), (1024, 8, 2, 0), (4096, 16, 3, 0), (4096, 3, 1, 1),
                                           (2048, 40, 2, 1)])
def test_march_equals_single_steps(n, M, nit, sched, prec):
    import paper_1101_0086_amd as P
    grid = Grid(n, 10.0 / 256)
    a = wdm_field(grid, n // 256, 1, "qpsk", np.random.default_rng(n + M))
    dmm = dm_map(beta3=0.1)
    L = 0.05
    say("one window", n, M, nit, sched, prec)
    plan = P.MPAPlan(n, grid.dt, dmm, L, M, nit, 0, 0, prec, schedule=sched)
    for m0, steps in ((0, 1), (8, 5), (17, 6)):            # within a span, across 0.5, across the amplifier at 1
        x, y = to_dev(a, prec), to_dev(a, prec)
        plan.propagate(x, m0 * L, (m0 + steps) * L)
        for m in range(m0, m0 + steps):
            plan.step(y, m * L)
        assert np.array_equal(to_host(x), to_host(y)), (m0, steps)
        ref = O.mpa_propagate(a, grid.dt, dmm, L, M, nit, m0 * L, (m0 + steps) * L)
        assert rel_l2(to_host(x), ref) < (TOL_F32 if prec == 0 else TOL_F64)
    plan.close()
