"""Reverse passes whose steps' forward recomputes share a launch (runs of four
or more steps with the same tables, few blocks) against the ones that do not
(store_steps = 2 never has four inputs at hand): bitwise the same gradient and
parameter derivatives, at step counts around the run lengths and with a span
change inside; and the oracle's gradient at the suite's tolerances."""
import math

import numpy as np
import pytest

import oracle as O
from tests.gpu_util import rel_l2, say, to_dev, to_host
from workloads import Grid, dm_map, wdm_field

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("block,M,nit,steps", [(512, 1, 1, 4), (512, 2, 2, 21), (1024, 3, 1, 5), (2048, 2, 2, 9),
                                               (4096, 1, 3, 7)])
def test_recompute_ahead(block, M, nit, steps, prec):
    import paper_1101_0086_amd as P
    n, dt, ch = 1 << 14, 10.0 / 1024, 4
    rng = np.random.default_rng(block + steps)
    a = wdm_field(Grid(n, dt), 16, ch, "qpsk", rng)
    target = wdm_field(Grid(n, dt), 16, ch, "qpsk", rng)     # content on the signal band
    dmm = dm_map(beta3=0.1)
    band, halo = 65.0, block // 4
    L = 0.5 / math.ceil(0.5 * O.halo_rate(band, 20.0, 0.1) / (0.24 * halo * dt))
    z0 = 0.5 - (steps // 3) * L                              # a span change inside the run
    z1 = z0 + steps * L
    say("adjoint ahead", block, M, nit, steps, prec)
    res = []
    for store in (0, 2):
        plan = P.MPAPlan(n, dt, dmm, L, M, nit, block, halo, prec, band)
        x = to_dev(a, prec)
        ck = plan.propagate_checkpointed(x, z0, z1)
        out = to_host(x)
        g = to_dev(2 * (out - target), prec)
        pg = plan.adjoint(ck, g, z0, z1, store)
        res.append((to_host(g), pg.cpu().numpy(), out))
        plan.close()
    assert np.array_equal(res[0][0], res[1][0]) and np.array_equal(res[0][1], res[1][1])
    g_out = 2 * (res[0][2] - target)
    gr, ds, d2, d3 = O.mpa_propagate_vjp(a, dt, dmm, L, M, nit, z0, z1, g_out, block=block, halo=halo)
    assert rel_l2(res[0][0], gr) < (1e-5 if prec == 0 else 1e-10)
    ref = np.concatenate([ds, d2, d3])
    assert np.linalg.norm(res[0][1].ravel() - ref) <= (1e-4 if prec == 0 else 1e-9) * np.linalg.norm(ref)
