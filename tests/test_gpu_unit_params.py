"""Bonded units of every split are laid out when the system is made, and follow gpr_set_params: forces and
energies after a change of parameters against the oracle (whose terms share no record with the
device's), on several ranges with terms inside and across, and shared launches that step with them
against the plain path, whatever split the launches take."""
import numpy as np
import pytest

import gpr_synth as G
import oracle
from test_gpu_small import _same, _spec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n", [("rl", 300), ("far", 601), ("chain", 513), ("chain", 40)])
def test_forces_after_set_params_match_oracle(kind, n):
    import paper_1807_02431_amd as gpr
    print("unit parameters", kind, n, flush=True)
    spec = G.round_to_f32(_spec(kind, n))
    s = gpr.System(spec, path=gpr.PATH_PERSISTENT)
    p = gpr.System(spec, path=gpr.PATH_PLAIN)
    rng = np.random.default_rng(n)
    for turn in range(2):
        new = {k: spec[k] * rng.uniform(0.7, 1.3, len(spec[k])) for k in ("epsilon", "sigma", "charge", "torsion_k")}
        for x in (s, p):
            x.set_params(**new)
        o = oracle.System(G.round_to_f32(dict(spec, **new)))
        E, F = p.energy_forces(0, 1)
        Uo, Fo = o.eval(p.get_state(0)[0])
        assert np.abs(F[0] - Fo).max() < 1e-5 * np.abs(Fo).max()
        assert abs(E[0] - Uo) <= 1e-5 * max(1.0, abs(Uo))
        for groups in (1, 2, 8, 4):
            s.set_launch(0, groups)
            gpr.batch_advance([s], 7)
            s.advance(6)
            p.advance(13)
            _same(s, p)
