"""Long steps of FP32 plans with one and two sweeps, whose node evaluations the
fused kernel runs in pairs, at the node counts where a pair is missing (one
node), left over (odd and even counts) and complete: bitwise the node-parallel
schedule, which runs every evaluation alone, and within the suite's FP32
tolerance of the oracle."""
import math

import numpy as np
import pytest

import oracle as O
from tests.gpu_util import TOL_F32, rel_l2, say, to_dev, to_host
from workloads import Grid, dm_map, wdm_field

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("block,nit", [(512, 1), (512, 2), (1024, 1), (2048, 2), (4096, 1), (4096, 2)])
def test_paired_evaluations(block, nit, M):
    import paper_1101_0086_amd as P
    n, dt, ch = 1 << 14, 10.0 / 1024, 4
    a = wdm_field(Grid(n, dt), 16, ch, "qpsk", np.random.default_rng(M))
    dmm = dm_map(beta3=0.1)
    band, halo = 65.0, block // 4 + 1              # odd halo, ragged last core
    L = 0.5 / math.ceil(0.5 * O.halo_rate(band, 20.0, 0.1) / (0.24 * halo * dt))
    z0, z1 = 0.5 - L, 0.5 + 2 * L                  # across the span change
    say("pairs", block, nit, M)
    got = []
    for sched in (P.MPA_WAVEFRONT, P.MPA_NODE_PARALLEL):
        plan = P.MPAPlan(n, dt, dmm, L, M, nit, block, halo, 0, band, schedule=sched)
        x = to_dev(a, 0)
        plan.propagate(x, z0, z1)
        got.append(to_host(x))
        plan.close()
    assert np.array_equal(got[0], got[1])
    ref = O.mpa_propagate(a, dt, dmm, L, M, nit, z0, z1, block, halo)
    assert rel_l2(got[0], ref) < TOL_F32
