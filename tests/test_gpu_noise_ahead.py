"""The persistent kernel draws the next step's Gaussians off the critical path where they have room in
LDS, and each step's own otherwise: both against the plain path, bit for bit, on both sides of that
rule (one group per replica holds the Gaussians up to about 1,600 atoms), with launches of one step,
rebuilds, samples and checks between."""
import numpy as np
import pytest

from test_gpu_small import _same, _spec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,bt,groups", [(161, 64, 1), (161, 1024, 8), (300, 256, 2), (301, 1024, 1), (1500, 1024, 1), (1650, 1024, 1),
                                         (1850, 512, 2), (3400, 1024, 4), (4600, 1024, 8)])
def test_gaussians_drawn_ahead_or_not(n, bt, groups):
    import paper_1807_02431_amd as gpr
    spec = dict(_spec("rl", n), n_replicas=2)
    print("noise ahead", n, bt, groups, flush=True)
    a = gpr.System(spec, path=gpr.PATH_PERSISTENT)
    a.set_launch(bt, groups)
    b = gpr.System(spec, path=gpr.PATH_PLAIN)
    for k in (1, 1, 2, 33):
        assert np.array_equal(a.advance(k), b.advance(k))
        _same(a, b)
