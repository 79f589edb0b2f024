"""What the library hands back through its page-locked buffer: states, accumulators, error flags and
first exit checks against each other over repeated calls, the most replicas a system takes,
calls that end at a check, between checks and without steps, and gradients whose
accumulators one call leaves clear for the next."""
import numpy as np
import pytest

import gpr_synth as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R,path", [(2, 0), (3, 1), (4096, 1), (4096, 0)])
def test_states_and_sums_of_many_replicas(R, path):
    import paper_1807_02431_amd as gpr
    print("read-back", R, path, flush=True)
    spec = G.toy2d(n_replicas=R, t_gr=3, t_check=10)
    a = gpr.System(spec, path=path)
    b = gpr.System(spec, path=path)
    fa = a.advance(30)                     # ends at a check; then the same steps in other pieces
    first = np.zeros(R, np.int64)
    for k in (5, 0, 7, 8, 10):             # between checks, none, across one, at one, at one
        f = b.advance(k)
        first = np.where(first == 0, f, first)
    assert np.array_equal(fa, first)
    na, A1, A2, sa = a.accumulators()
    nb, B1, B2, sb = b.accumulators()
    assert na == nb == 10 and np.array_equal(A1, B1) and np.array_equal(A2, B2) and np.array_equal(sa, sb)
    assert A1.shape[0] == R and np.all(A1[1:] != 0)
    for r in (0, 1, R // 2, R - 1):
        for x, y in zip(a.get_state(r), b.get_state(r)):
            assert np.array_equal(x, y)
    q, v = a.get_state(R - 1)
    a.set_state(R - 1, q + 0.25, v * 2.0)
    q2, v2 = a.get_state(R - 1)
    assert np.array_equal(q2[:2], (q + 0.25).astype(np.float32)[:2]) and np.array_equal(v2[:2], (v * 2.0).astype(np.float32)[:2])


def test_gradients_repeat():
    import torch

    from paper_1807_02431_amd.autograd import EnergyModel
    spec = G.chain(n_atoms=22, n_replicas=3, t_check=50)
    m = EnergyModel(spec)
    pos = torch.tensor(spec["pos"], dtype=torch.float32, device="cuda").expand(3, 3, 22).contiguous()
    ref = None
    for turn in range(4):
        host = turn == 2                   # parameters that stay on the host take no gradients
        leaves = [pos.clone().requires_grad_()] + [p if host else p.requires_grad_() for p in m.parameters("cpu" if host else "cuda")]
        U = m(*leaves)
        wants = leaves[:1] if host else leaves[:1] + leaves[2:3] if turn == 1 else leaves
        g = [x.cpu() for x in torch.autograd.grad(U.sum(), wants)]
        if len(wants) < 5:
            assert torch.equal(g[0], ref[1][0]) and (host or torch.equal(g[1], ref[1][2]))
            continue
        if ref is None:
            ref = (U.detach().cpu(), g)
        assert torch.equal(U.detach().cpu(), ref[0])
        assert all(torch.equal(a, b) for a, b in zip(g, ref[1]))
