"""The autotuner leaves no system slower than the shape its launches take by themselves, which for few
replicas has more workgroups than the shapes it tries."""
import time

import pytest

from test_gpu_small import _same, _spec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n,R", [("rl", 2432, 2), ("chain", 22, 64)])
def test_tuned_is_not_slower_than_untuned(kind, n, R):
    import paper_1807_02431_amd as gpr
    print("autotune", kind, n, R, flush=True)
    spec = dict(_spec(kind, n), n_replicas=R, t_check_dephase=2000)
    a, b = (gpr.System(spec, path=gpr.PATH_PERSISTENT) for _ in range(2))
    bt, g = a.autotune(200)
    assert bt in (256, 512, 768, 1024) and g in (1, 2, 4, 8)
    took = []
    for s in (a, b):
        t = []
        for _ in range(9):
            t0 = time.perf_counter()
            s.advance(400)
            t.append(time.perf_counter() - t0)
        took.append(min(t))
    print("tuned", took[0], "untuned", took[1], flush=True)
    assert took[0] < 1.2 * took[1]         # (12.7 against 9.2 us a step before, and the runs of one side differ by 1 %)
    _same(a, b)
