"""FP64 rounding of the one-workgroup split-step's transforms: with no
dispersion, nonlinearity and loss a step is a transform and its inverse (their
scale a power of two), so what is left after 64 steps is their rounding.  The
bounds are the values of transforms whose twiddles all come from the table,
measured on these inputs with products of seven of them; with the
e^{i pi/4} w of a pass formed from w they are exceeded by 4 to 18 %."""
import numpy as np
import pytest

from tests.gpu_util import say, to_dev, to_host

pytestmark = pytest.mark.gpu


class _Nothing:
    seg_len = (0.5, 0.5)
    beta2 = beta3 = sigma = (0.0, 0.0)
    gamma = z_amp = raman_g0 = raman_alpha = 0.0


@pytest.mark.parametrize("n,bound", [(512, 1.442e-14), (1024, 1.535e-14), (2048, 1.686e-14), (4096, 1.847e-14)])
def test_round_trips(n, bound):
    import paper_1101_0086_amd as P
    rng = np.random.default_rng(n)
    dz = 0.5 / 1024
    total = 0.0
    for k in range(4):
        a = rng.normal(size=n) + 1j * rng.normal(size=n)
        say("round trips", n, k)
        plan = P.SSPlan(n, 10.0 / 256, _Nothing(), dz, P.MPA_C128)
        x = to_dev(a, 1)
        plan.propagate(x, 0.0, 64 * dz)
        total += np.linalg.norm(to_host(x) - a) ** 2 / np.linalg.norm(a) ** 2
        plan.close()
    assert np.sqrt(total / 4) < bound
