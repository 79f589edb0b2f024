"""The parameter gradient at the positions that a stepping call or a copy of replicas left, without an
evaluation in between: the pair lists it runs over are those of these positions.  The reference is
the same call after an evaluation at the same positions (which rebuilds every list); the sums are
fixed point and pairs beyond the cutoff add exact zeros, so the two agree bit for bit."""
import numpy as np
import pytest

from test_gpu_small import _spec

pytestmark = pytest.mark.gpu


def _gradient(s):
    import torch
    w = torch.linspace(0.5, 1.5, s.R, dtype=torch.float64, device="cuda")
    out = [torch.empty(k, dtype=torch.float64, device="cuda") for k in (s.n, s.n, s.n, max(1, s.nt))]
    dx = torch.empty((s.R, 3, s.n), dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    s.energy_backward_dev(w.data_ptr(), dx.data_ptr(), *(t.data_ptr() for t in out))
    return [dx.cpu().numpy()] + [t.cpu().numpy() for t in out]


@pytest.mark.parametrize("n,then", [(80, "steps"), (160, "steps"), (161, "steps"), (160, "copies"), (300, "copies"), (120, "cycles")])
def test_gradient_after_steps_and_copies(n, then):
    import torch
    import paper_1807_02431_amd as gpr
    print("gradient lists", n, then, flush=True)
    spec = dict(_spec("rl", n), t_check_dephase=500)
    s = gpr.System(spec, path=gpr.PATH_PERSISTENT, stream=torch.cuda.current_stream())
    s.advance(5000)
    if then == "copies":
        s.set_path(gpr.PATH_PLAIN)
        s.dephase(max_steps=0)             # every replica takes the reference walker's positions
    elif then == "cycles":
        s.set_cycles(2)
        s.dephase(max_steps=1000)
    got = _gradient(s)
    x = torch.tensor(np.stack([s.get_state(r)[0] for r in range(s.R)]).astype(np.float32), device="cuda")
    torch.cuda.synchronize()
    s.energy_forces_dev(x.data_ptr(), 0, 0)
    for a, b in zip(got, _gradient(s)):
        assert np.array_equal(a, b)
