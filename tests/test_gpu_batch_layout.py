"""Shared and single launches over replica counts that are no multiple of eight, that take the sets
several rounds, and mixes in which the layout changes a system's workgroups per replica: the same
states as each system alone on one workgroup per replica, bit for bit."""
import numpy as np
import pytest

from test_gpu_small import _same, _spec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mix", [[("rl", 300, 12)], [("rl", 600, 9), ("toy", 1, 5)], [("rl", 1200, 60)],
                                 [("chain", 22, 300), ("rl", 300, 70), ("rl", 1200, 40), ("chain", 300, 3)],
                                 [("rl", 2432, 17), ("rl", 161, 100)], [("rl", 4600, 9), ("rl", 300, 11)]])
def test_layouts_match_single_systems(mix):
    import paper_1807_02431_amd as gpr
    print("batch layout", mix, flush=True)
    specs = [dict(_spec(k, n), n_replicas=R, t_check_dephase=20) for k, n, R in mix]
    together = [gpr.System(s, path=gpr.PATH_PERSISTENT) for s in specs]
    alone = [gpr.System(s, path=gpr.PATH_PERSISTENT) for s in specs]
    own = [gpr.System(s, path=gpr.PATH_PERSISTENT) for s in specs]
    for (k, n, R), s in zip(mix, own):
        s.set_launch(256 if n < 1000 else 0, 1 if n < 1500 else 8)      # the caller's shape stays
    for k in (1, 30, 14):
        ft = gpr.batch_advance(together, k)
        fo = gpr.batch_advance(own, k)
        for a, f, g in zip(alone, ft, fo):
            h = a.advance(k)
            assert np.array_equal(f, h) and np.array_equal(g, h)
    for t, o, a in zip(together, own, alone):
        _same(t, a)
        _same(o, a)
