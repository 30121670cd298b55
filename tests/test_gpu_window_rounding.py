"""FP32 rounding of windows above 4096 modes: one strongly nonlinear long step
(sigma L times the mean power 0.5, so that the node transforms' rounding and
not the stored field's decides) against the same step in FP64.  The bounds are
the errors of transforms that multiply every input of a pass by its own rounded
twiddle, measured on these inputs (1.444e-7, 1.649e-7 and 1.886e-7), plus 2 %;
transforms whose passes apply three rounded twiddles in a row are 7 to 12 %
above them."""
import numpy as np
import pytest

from tests.gpu_util import rel_l2, say, to_dev, to_host
from workloads import Grid, dm_map
from workloads.wdm import _fast_wdm_field

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lg,measured", [(13, 1.444e-7), (16, 1.649e-7), (18, 1.886e-7)])
def test_fp32_window_rounding(lg, measured):
    import paper_1101_0086_amd as P
    n, dt, L = 1 << lg, 10.0 / 1024, 2.5e-4
    a = _fast_wdm_field(Grid(n, dt), n // 1024, 8, "qpsk", np.random.default_rng(5)).astype(np.complex64)
    dmm = dm_map(beta3=0.1, sigma=0.5 / (L * float(np.mean(np.abs(a) ** 2))))
    out = []
    for prec in (0, 1):
        say("window rounding", lg, prec)
        plan = P.MPAPlan(n, dt, dmm, L, 1, 1, 0, 0, prec)
        x = to_dev(a, prec)
        plan.propagate(x, 0.0, L)
        out.append(to_host(x))
        plan.close()
    assert rel_l2(out[0], out[1]) < 1.02 * measured
