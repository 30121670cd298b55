"""Strongly nonlinear split-steps: the kick exp(i sigma |A|^2 dz) with phases
around the bounds of its forms (1/64, 2^20) and far between them, against the
oracle; and its cost, which stays near that of the transforms around it.

One step, so that the error of a phase is not amplified by the next kick: the
phase's own rounding and that of the field it is formed from are a few 1e-16
of the phase, and the suite's tolerances hold up to phases of 1e3 in FP64;
beyond, 2e-14 of the phase.  FP32 fields are the same arithmetic on a rounded
input."""
import numpy as np
import pytest

import oracle as O
from tests.gpu_util import TOL_F64, rel_l2, say, to_dev, to_host, torch_mod
from workloads import Grid, dm_map, wdm_field

pytestmark = pytest.mark.gpu

DZ = 1.0 / 320


def _plan(n, prec, peak):
    import paper_1101_0086_amd as P
    grid = Grid(n, 10.0 / 256)
    a = wdm_field(grid, n // 256, 1, "qpsk", np.random.default_rng(n))
    if prec == 0:
        a = a.astype(np.complex64).astype(np.complex128)
    sigma = peak / (DZ * float(np.max(np.abs(a)) ** 2))
    dmm = dm_map(beta3=0.0, sigma=sigma)
    return a, grid, dmm, P.SSPlan(n, grid.dt, dmm, DZ, prec)


@pytest.mark.parametrize("n", [512, 2048, 4096, 16384])
@pytest.mark.parametrize("peak", [0.03, 0.8, -1.6, 30.0, -1e3, 1e5, 1.2e6, -4e6])
def test_strong_kick(n, peak):
    a, grid, dmm, plan = _plan(n, 1, peak)
    say("strong kick", n, peak)
    x = to_dev(a, 1)
    plan.propagate(x, 0.0, DZ)
    plan.close()
    ref = O.ss_propagate(a, grid.dt, dmm, DZ, 0.0, DZ)
    assert rel_l2(to_host(x), ref) < max(TOL_F64, 2e-14 * abs(peak))


@pytest.mark.parametrize("n,prec", [(512, 1), (1024, 0), (2048, 1), (4096, 1)])
def test_strong_kick_costs_little_more(n, prec):
    """A run whose every kick lies beyond the polynomial of small phases takes
    at most 1.6 times a weakly nonlinear one's time.  Forming sin and cos of
    eight points one after another took 2.0 to 2.3 times; the reduced
    polynomials are about 40 operations a point beside the transforms' 250."""
    torch = torch_mod()
    us = {}
    for peak in (1.0 / 256, 1.0 / 32, 2.0):
        a, _, _, plan = _plan(n, prec, peak)
        x = to_dev(a, prec)
        say("kick time", n, prec, peak)
        times = []
        for _ in range(12):
            t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            t0.record()
            plan.propagate(x, 0.0, 128 * DZ)
            t1.record()
            t1.synchronize()
            times.append(t0.elapsed_time(t1))
        plan.close()
        us[peak] = sorted(times)[len(times) // 2]
    assert max(us.values()) <= 1.6 * us[1.0 / 256], us
