"""The position exchange between the workgroups of a replica: launches longer than its tags count
(32,767 steps), groups without atoms, atom counts around a pass of the polling threads, and many short
launches in a row over the same buffers, against one group per replica, bit for bit."""
import numpy as np
import pytest

from test_gpu_small import _same, _spec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n,bt,groups,chunks", [("chain", 258, 256, 2, (33000, 1)), ("chain", 258, 64, 8, (1,) * 20 + (2,) * 20),
                                                     ("rl", 161, 64, 8, (3, 1, 40)), ("rl", 170, 1024, 4, (3, 1, 40)),
                                                     ("rl", 1200, 128, 8, (2, 1, 30)), ("rl", 1500, 512, 2, (2, 1, 30))])
def test_exchange_matches_one_group(kind, n, bt, groups, chunks):
    import paper_1807_02431_amd as gpr
    spec = dict(_spec(kind, n), t_check_dephase=40000, n_replicas=9 if n < 300 else 2)
    print("exchange", kind, n, bt, groups, flush=True)
    a = gpr.System(spec, path=gpr.PATH_PERSISTENT)
    a.set_launch(bt, groups)
    b = gpr.System(spec, path=gpr.PATH_PERSISTENT)
    b.set_launch(512, 1)
    for k in chunks:
        a.advance(k)
    b.advance(sum(chunks))
    _same(a, b)


@pytest.mark.parametrize("n,R", [(1024, 2), (1100, 5), (2047, 3), (2100, 8), (4600, 2)])
def test_many_groups_for_few_replicas(n, R):
    """Launches of few replicas take up to 32 workgroups each by themselves: the same walker, states and
    samples as on the caller's shape."""
    import paper_1807_02431_amd as gpr
    spec = dict(_spec("rl", n), n_replicas=R, t_check_dephase=20)
    print("many groups", n, R, flush=True)
    a = gpr.System(spec, path=gpr.PATH_PERSISTENT)
    b = gpr.System(spec, path=gpr.PATH_PERSISTENT)
    b.set_launch(1024, 8)
    for _ in range(2):
        assert a.decorrelate(40, max_steps=40) == b.decorrelate(40, max_steps=40)
        assert np.array_equal(a.advance(25), b.advance(25))
    _same(a, b)
