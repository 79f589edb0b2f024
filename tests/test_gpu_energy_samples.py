"""The potential energy as an observable on every step, its sum over a replica's workgroups cleared and added
to again from one step to the next: the plain path's accumulators, bit for bit, over long launches."""
import numpy as np
import pytest

import gpr_synth as G
from test_gpu_small import _same, _spec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,groups,R", [(161, 2, 3), (300, 8, 24), (1200, 8, 4), (2432, 0, 2)])
def test_energy_sampled_on_every_step(n, groups, R):
    import paper_1807_02431_amd as gpr
    print("energy samples", n, groups, R, flush=True)
    spec = dict(_spec("rl", n), n_replicas=R, t_gr=1, t_check_dephase=1000, obs=[dict(kind=G.OBS_POTENTIAL), dict(kind=G.OBS_KINETIC)])
    a = gpr.System(spec, path=gpr.PATH_PERSISTENT)
    if groups:
        a.set_launch(0, groups)
    b = gpr.System(spec, path=gpr.PATH_PLAIN)
    for k in (1, 400, 99):
        a.advance(k)
        b.advance(k)
        _same(a, b)
