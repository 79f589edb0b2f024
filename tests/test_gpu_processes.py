"""Two processes on one device, whose launches each ask for more than half of it and wait for their own workgroups:
both end, with the results of a process that runs alone."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

_CHILD = r"""
import sys
sys.path.insert(0, %(root)r)
sys.path.insert(0, %(root)r + "/tests")
import hashlib
import numpy as np
import paper_1807_02431_amd as gpr
from test_gpu_small import _spec
h = hashlib.sha256()
for n, R in ((300, 24), (2432, 64), (1200, 8)):
    s = gpr.System(dict(_spec("rl", n), n_replicas=R, t_check_dephase=20), path=gpr.PATH_PERSISTENT)
    for k in range(30):
        h.update(np.asarray(s.advance(10 + k)).tobytes())
    for r in range(R):
        for x in s.get_state(r):
            h.update(x.tobytes())
print(h.hexdigest())
"""


def _start():
    return subprocess.Popen([sys.executable, "-c", _CHILD % dict(root=ROOT)], stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True)


def _end(p):
    out, err = p.communicate(timeout=100)
    assert p.returncode == 0, err[-2000:]
    return out.strip().splitlines()[-1]


def test_two_processes_share_the_device():
    print("two processes", flush=True)
    alone = _end(_start())
    both = [_start(), _start()]
    assert [_end(p) for p in both] == [alone, alone]
