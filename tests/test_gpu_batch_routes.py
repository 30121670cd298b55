"""An instance of a batch (always the fused kernel) against a plan of its own
whose few blocks and many nodes run on the node-parallel kernels: bitwise the
same field, and bitwise the same gradient, in both precisions, with one to
four blocks per field, one to three sweeps, and sums of Eq. 6 added by the
nodes' workgroups or in launches of their own (M x block >= 65536).  Both
perform the same operations in the same order, so nothing may differ; the
oracle at the suite's tolerances."""
import math

import numpy as np
import pytest

import oracle as O
from tests.gpu_util import TOL_F32, TOL_F64, rel_l2, say, to_dev, to_host
from workloads import Grid, dm_map, wdm_field

pytestmark = pytest.mark.gpu

DT = 10.0 / 1024
CASES = [(512, 5, 1, 1), (1024, 4, 2, 1), (2048, 4, 3, 1), (4096, 4, 2, 1), (4096, 16, 3, 1), (2048, 40, 1, 1),
         (512, 9, 1, 0), (1024, 8, 2, 0), (2048, 8, 3, 0), (4096, 16, 3, 0)]


def _case(block, M):
    ns = [max(block, 1024), 2 * max(block, 1024)]
    rng = np.random.default_rng(block + M)
    fields = [wdm_field(Grid(n, DT), n // 1024, 4, "qpsk", rng) for n in ns]
    halo = block // 8
    k = math.ceil(0.5 * O.halo_rate(65.0, 20.0, 0.1) / (0.24 * halo * DT))
    return ns, fields, halo, 0.5 / k


@pytest.mark.parametrize("block,M,nit,prec", CASES)
def test_batch_instance_is_its_own_plan(block, M, nit, prec):
    import paper_1101_0086_amd as P
    ns, fields, halo, L = _case(block, M)
    scales = [1.0, 1.7]
    dmm = dm_map(beta3=0.1)
    z0, z1 = 0.5 - 2 * L, 0.5 + 2 * L                  # across the span change
    say("batch against own plan", block, M, nit, prec)
    bp = P.MPABatchPlan(ns, DT, dmm, L, M, nit, block, halo, prec, 65.0, sigma_scale=scales)
    x = to_dev(np.concatenate(fields), prec)
    ck = bp.propagate_checkpointed(x, z0, z1)
    got = [to_host(v) for v in bp.split(x)]
    g = to_dev(np.concatenate([0.5 * a for a in fields]), prec)
    bp.adjoint(ck, g, z0, z1)
    grads = [to_host(v) for v in bp.split(g)]
    bp.close()
    for a, n, sc, field, grad in zip(fields, ns, scales, got, grads):
        p = P.MPAPlan(n, DT, dmm.with_sigma(sc), L, M, nit, block, halo, prec, 65.0)
        info = p.info()
        assert info["workspace_bytes"] > n * (8 if prec == 0 else 16)      # runs on the node-parallel kernels
        y = to_dev(a, prec)
        p.propagate(y, z0, z1)
        assert np.array_equal(to_host(y), field), (n, info["n_blocks"])
        y = to_dev(a, prec)
        ck = p.propagate_checkpointed(y, z0, z1)
        assert np.array_equal(to_host(y), field)
        g = to_dev(0.5 * a, prec)
        p.adjoint(ck, g, z0, z1)
        assert np.array_equal(to_host(g), grad), (n, info["n_blocks"])
        p.close()
        ref = O.mpa_propagate(a, DT, dmm.with_sigma(sc), L, M, nit, z0, z1, block, halo)
        assert rel_l2(field, ref) < (TOL_F32 if prec == 0 else TOL_F64)
