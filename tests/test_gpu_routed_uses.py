"""Default-schedule plans that run on the node-parallel kernels (few blocks,
many nodes) in the other uses of a plan: captured and replayed, as the forward
of a gradient whose step inputs are recomputed on a second stream, kept, or
recomputed one by one (bitwise the same), and in the Picard residuals."""
import math

import numpy as np
import pytest

import oracle as O
from tests.gpu_util import rel_l2, say, to_dev, to_host
from workloads import Grid, dm_map, wdm_field

pytestmark = pytest.mark.gpu

DT = 10.0 / 1024


def _plan(kind, M, nit, prec):
    import paper_1101_0086_amd as P
    if kind == "window":
        n, dt, block, halo, band, L = 1024, 10.0 / 256, 0, 0, 0.0, 0.05
        a = wdm_field(Grid(n, dt), 4, 1, "qpsk", np.random.default_rng(M))
    else:
        n, dt, block, halo, band = 8192, DT, 2048, 256, 65.0
        a = wdm_field(Grid(n, dt), 8, 4, "qpsk", np.random.default_rng(M))
        L = 0.5 / math.ceil(0.5 * O.halo_rate(band, 20.0, 0.1) / (0.24 * halo * dt))
    plan = P.MPAPlan(n, dt, dm_map(beta3=0.1), L, M, nit, block, halo, prec, band)
    assert plan.info()["workspace_bytes"] > n * (8 if prec == 0 else 16)
    return plan, a, L


@pytest.mark.parametrize("kind,M,nit,prec", [("window", 16, 2, 0), ("window", 70, 2, 1), ("blocks", 8, 1, 0),
                                             ("blocks", 5, 2, 1)])
def test_captured_march(kind, M, nit, prec):
    import torch
    plan, a, L = _plan(kind, M, nit, prec)
    say("captured routed march", kind, M, nit, prec)
    g, e = to_dev(a, prec), to_dev(a, prec)
    graph = plan.capture(g, 0.5 - 2 * L, 0.5 + L)
    other = torch.zeros(1 << 16, device="cuda:0")
    for rep in range(4):
        graph.launch()
        plan.propagate(e, 0.5 - 2 * L, 0.5 + L)
        other.add_(1.0)
        torch.cuda.synchronize()
        assert np.array_equal(to_host(g), to_host(e)), rep
    graph.close()
    plan.close()


@pytest.mark.parametrize("kind,M,nit,prec", [("window", 8, 2, 0), ("window", 4, 3, 1), ("blocks", 8, 2, 0),
                                             ("blocks", 4, 2, 1)])
def test_gradient_over_period_boundaries(kind, M, nit, prec):
    plan, a, L = _plan(kind, M, nit, prec)
    say("gradient of a routed plan", kind, M, nit, prec)
    z0, z1 = 1.0 - 5 * L, 1.0 + 6 * L              # two segments: the second recomputed beside the first's reverse
    target = to_dev(0.5 * a, prec)
    got = []
    for keep, store in ((0, 0), (1 << 30, 0), (0, 1)):
        plan.keep_inputs(keep)
        x = to_dev(a, prec)
        ck = plan.propagate_checkpointed(x, z0, z1)
        assert ck.shape[0] == 2
        g = (2 * (x - target)).contiguous()
        pg = plan.adjoint(ck, g, z0, z1, store)
        got.append((to_host(x), to_host(g), pg.cpu().numpy()))
    y = to_dev(a, prec)
    plan.propagate(y, z0, z1)
    plan.close()
    assert np.array_equal(to_host(y), got[0][0])
    for other in got[1:]:
        for u, v in zip(got[0], other):
            assert np.array_equal(u, v)


@pytest.mark.parametrize("prec", [0, 1])
def test_picard_residuals(prec):
    """Against the fused kernel (the allocation-free march with k sweeps)."""
    import paper_1101_0086_amd as P
    n, dt, L, M, nit = 1024, 10.0 / 256, 0.05, 16, 3
    plan, a, _ = _plan("window", M, nit, prec)
    dmm = dm_map(beta3=0.1)
    say("residuals of a routed plan", prec)
    st, r = plan.picard_residuals(to_dev(a, prec), 0.2, nit)
    plan.close()
    outs = []
    for sweeps in range(1, nit + 1):
        x = to_dev(a, prec)
        outs.append(to_host(P.propagate_noalloc(x, dt, dmm, L, M, sweeps, 0.2, 0.2 + L, precision=prec)))
    for k in (2, 3):
        want = np.linalg.norm(outs[k - 1] - outs[k - 2]) / np.linalg.norm(outs[k - 1])
        assert abs(r[k - 1] - want) <= (1e-6 if prec == 0 else 1e-12), (k, r, want)
