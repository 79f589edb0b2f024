"""Masses between those of the light and the heavy margin class: states do not depend on when lists are rebuilt
(by the margins, or on every step), bit for bit, on both paths."""
import numpy as np
import pytest

from test_gpu_small import _same, _spec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("masses", [(1.0, 2.5, 16.0), (1.0, 3.99, 4.0), (3.0, 7.0, 11.0), (2.0, 9.0, 400.0)])
def test_margins_of_middle_masses(masses):
    import paper_1807_02431_amd as gpr
    print("margins", masses, flush=True)
    spec = _spec("rl", 300)
    spec["mass"] = np.random.default_rng(5).choice(masses, 300).astype(np.float64)
    spec["nlist_period"] = 1000
    sys = [gpr.System(spec, path=gpr.PATH_PERSISTENT), gpr.System(spec, path=gpr.PATH_PLAIN),
           gpr.System(dict(spec, nlist_period=1), path=gpr.PATH_PLAIN)]
    for k in (1, 200, 150):
        for s in sys:
            s.advance(k)
        _same(sys[0], sys[2])
        _same(sys[1], sys[2])
