"""Handles stepped from several threads on streams of their own, whose launches each ask for much of the device
(replicas over several workgroups that wait for one another): every call ends, with the results of
the same calls one after the other, bit for bit."""
import threading

import numpy as np
import pytest

from test_gpu_small import _same, _spec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mix", [[("rl", 300, 24), ("rl", 300, 24), ("rl", 400, 20)],
                                 [("rl", 2432, 64), ("rl", 300, 24), ("rl", 2432, 4)],
                                 [("rl", 1200, 8), ("rl", 1200, 40), ("toy", 1, 8), ("rl", 2432, 2)]])
def test_overlapping_calls_end_and_agree(mix):
    import torch
    import paper_1807_02431_amd as gpr
    print("streams", mix, flush=True)
    specs = [dict(_spec(k, n), n_replicas=R, t_check_dephase=25) for k, n, R in mix]
    alone = [gpr.System(s, path=gpr.PATH_PERSISTENT) for s in specs]
    streams = [torch.cuda.Stream() for _ in mix]
    together = [gpr.System(s, path=gpr.PATH_PERSISTENT, stream=st) for s, st in zip(specs, streams)]
    together[0].set_cycles(2)
    alone[0].set_cycles(2)

    def work(s, out):
        try:
            for k in (10, 40, 25):
                out.append(s.advance(k))
                out.append(s.decorrelate(50, max_steps=50))
            out.append(s.dephase(max_steps=60)[0])
        except Exception as e:              # (reported by the main thread)
            out.append(e)

    got = [[] for _ in mix]
    threads = [threading.Thread(target=work, args=(s, o)) for s, o in zip(together, got)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for s, t, o in zip(alone, together, got):
        ref = []
        work(s, ref)
        assert not [e for e in ref + o if isinstance(e, Exception)]
        for a, b in zip(ref, o):
            assert np.array_equal(a, b) if isinstance(a, np.ndarray) else a == b
        _same(s, t)
