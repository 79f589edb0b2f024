"""Replicas of fewer blocks of 16 atoms than the workgroups asked for (the toy on 2, chains on 2 to 8), sampled on
every step over long launches, and the autotuner on them: the plain path's states, sums and exit
checks, bit for bit."""
import numpy as np
import pytest

from test_gpu_small import _same, _spec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n,bt,groups", [("toy", 1, 64, 2), ("toy", 1, 64, 8), ("chain", 14, 64, 2), ("chain", 22, 64, 8),
                                              ("chain", 33, 128, 4), ("rl", 100, 256, 8)])
def test_tiny_replicas_on_many_groups(kind, n, bt, groups):
    import paper_1807_02431_amd as gpr
    print("tiny replicas", kind, n, bt, groups, flush=True)
    spec = dict(_spec(kind, n), t_gr=1, t_check_dephase=700)
    a = gpr.System(spec, path=gpr.PATH_PERSISTENT)
    a.set_launch(bt, groups)
    b = gpr.System(spec, path=gpr.PATH_PLAIN)
    for k in (1, 2, 1500):
        assert np.array_equal(a.advance(k), b.advance(k))
        _same(a, b)
    a.autotune(20)
    assert np.array_equal(a.advance(150), b.advance(150))
    _same(a, b)
