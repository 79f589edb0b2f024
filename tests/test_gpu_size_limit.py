"""The largest system the plain path takes: 6,136 atoms fill a workgroup's LDS (24 bytes an atom of a padded
6,144, 16 a block of eight, 4 KB of search scratch, 16 static) to the byte.  Forces match the oracle
there and at the first size of the last padding step; one atom more is refused as too large."""
import numpy as np
import pytest

import gpr_synth as G
import oracle

pytestmark = pytest.mark.gpu


def _spec(n):
    return G.round_to_f32(G.receptor_ligand(n_receptor=n - 32, radius=5.6, n_replicas=2))


@pytest.mark.parametrize("n", [6080, 6136])
def test_largest_plain_system(n):
    import paper_1807_02431_amd as gpr
    print("largest plain system", n, flush=True)
    spec = _spec(n)
    g = gpr.System(spec)
    g.advance(12)                          # (a period's rebuild among them)
    E, F = g.energy_forces()
    o = oracle.System(spec)
    for r in range(2):
        Uo, Fo = o.eval(g.get_state(r)[0])
        assert np.abs(F[r] - Fo).max() < 1e-5 * np.abs(Fo).max()
        assert abs(E[r] - Uo) <= 1e-5 * abs(Uo)


def test_one_atom_more_is_refused():
    import paper_1807_02431_amd as gpr
    print("one atom more", flush=True)
    with pytest.raises(gpr.GprError) as e:
        gpr.System(_spec(6137))
    assert e.value.code == -1
