"""The node-parallel kernels' launch forms against the fused kernel, bitwise in
both precisions, and against the oracle at the suite's tolerances.  Each
comparison makes sure of its two sides: plans with the wavefront schedule run
the fused kernel when n_blocks > 4 M (their workspace is then one field), and
batches always do.

  many     more blocks than CUs: U_0 computed with psi_0, node numbering from
           one, one exchange buffer throughout; odd last core
  shared   a few hundred node workgroups (one exchange buffer in the sweeps,
           U_0 as node 0)
  summed   sums of Eq. 6 in launches of their own, two to four blocks
  fused    the fused kernel's FP64 and three to five sweep forms at 4 < M"""
import math

import numpy as np
import pytest

import oracle as O
from tests.gpu_util import TOL_F32, TOL_F64, rel_l2, say, to_dev, to_host
from workloads import Grid, dm_map, wdm_field

pytestmark = pytest.mark.gpu

DT = 10.0 / 1024


def _case(n, halo, seed):
    a = wdm_field(Grid(n, DT), n // 1024, 4, "qpsk", np.random.default_rng(seed))
    k = math.ceil(0.5 * O.halo_rate(65.0, 20.0, 0.1) / (0.24 * halo * DT))
    return a, dm_map(beta3=0.1), 0.5 / k


def _march(plan, a, prec, z0, z1):
    x = to_dev(a, prec)
    plan.propagate(x, z0, z1)
    out = to_host(x)
    plan.close()
    return out


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("form,n,block,halo,M,nit", [
    ("many", 1 << 17, 512, 37, 1, 2), ("many", 1 << 17, 512, 37, 2, 1), ("many", 1 << 18, 1024, 129, 2, 3),
    ("shared", 1 << 15, 512, 128, 3, 2), ("shared", 1 << 16, 2048, 256, 5, 1), ("shared", 1 << 18, 4096, 512, 4, 2),
    ("fused", 1 << 14, 512, 64, 5, 4), ("fused", 1 << 15, 1024, 128, 6, 5), ("fused", 1 << 17, 4096, 512, 7, 3)])
def test_against_the_fused_kernel(form, n, block, halo, M, nit, prec):
    import paper_1101_0086_amd as P
    a, dmm, L = _case(n, halo, n + M)
    z0, z1 = 0.5 - L, 0.5 + 2 * L                      # across the span change
    args = (n, DT, dmm, L, M, nit, block, halo, prec, 65.0)
    say("schedule paths", form, n, block, M, nit, prec)
    fused, nodes = P.MPAPlan(*args), P.MPAPlan(*args, schedule=P.MPA_NODE_PARALLEL)
    field = n * (8 if prec == 0 else 16)
    nb = fused.info()["n_blocks"]
    assert fused.info()["workspace_bytes"] == field and nodes.info()["workspace_bytes"] > field
    assert {"many": nb > 256, "shared": nb <= 256 < nb * (M + 1), "fused": nb > 4 * M}[form], nb
    got = _march(nodes, a, prec, z0, z1)
    assert np.array_equal(_march(fused, a, prec, z0, z1), got)
    ref = O.mpa_propagate(a, DT, dmm, L, M, nit, z0, z1, block, halo)
    assert rel_l2(got, ref) < (TOL_F32 if prec == 0 else TOL_F64)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n,block,halo,M,nit", [(1 << 12, 4096, 512, 16, 3), (1 << 13, 4096, 512, 16, 3),
                                                (1 << 13, 4096, 1024, 16, 1), (1 << 13, 4096, 512, 23, 2)])
def test_sums_of_their_own(n, block, halo, M, nit, prec):
    import paper_1101_0086_amd as P
    a, dmm, L = _case(n, halo, n + M)
    z0, z1 = 0.5 - L, 0.5 + 2 * L
    say("sums apart", n, M, nit, prec)
    plan = P.MPAPlan(n, DT, dmm, L, M, nit, block, halo, prec, 65.0)
    info = plan.info()
    assert info["workspace_bytes"] > n * (8 if prec == 0 else 16) and 2 <= info["n_blocks"] <= M * block // 16384
    got = _march(plan, a, prec, z0, z1)
    batch = P.MPABatchPlan([n], DT, dmm, L, M, nit, block, halo, prec, 65.0)
    assert np.array_equal(_march(batch, a, prec, z0, z1), got)
    ref = O.mpa_propagate(a, DT, dmm, L, M, nit, z0, z1, block, halo)
    assert rel_l2(got, ref) < (TOL_F32 if prec == 0 else TOL_F64)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n,M,nit", [(512, 16, 2), (4096, 16, 3), (2048, 9, 5)])
def test_one_window_against_the_allocation_free_march(n, M, nit, prec):
    """One full window: the plan runs node-parallel, the allocation-free march
    the fused kernel on tables built on the device (the same to the last bits:
    1e-13 of the field in FP64 after three steps, three FP32 roundings of it
    and of the tables in FP32)."""
    import paper_1101_0086_amd as P
    dt, L = 10.0 / 256, 0.05
    a = wdm_field(Grid(n, dt), n // 256, 1, "qpsk", np.random.default_rng(n))
    dmm = dm_map(beta3=0.1)
    say("one window", n, M, nit, prec)
    plan = P.MPAPlan(n, dt, dmm, L, M, nit, 0, 0, prec)
    assert plan.info()["workspace_bytes"] > n * (8 if prec == 0 else 16)
    got = _march(plan, a, prec, 8 * L, 11 * L)
    x = to_dev(a, prec)
    P.propagate_noalloc(x, dt, dmm, L, M, nit, 8 * L, 11 * L, precision=prec)
    assert rel_l2(to_host(x), got) < (1e-6 if prec == 0 else 1e-13)
