"""The bonded units of the persistent kernel (64 terms of one kind, by atom range) against the plain
path, which takes a term per thread, bit for bit: one to eight ranges, terms inside a range and
across, neighbours far apart in index, unit counts around a multiple of 64, and parameters that
change before the units are first laid out, after, and for a split that is laid out later."""
import numpy as np
import pytest

from test_gpu_small import _same, _spec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,n,groups", [("rl", 161, 1), ("rl", 161, 8), ("far", 170, 2), ("far", 300, 8), ("far", 301, 1),
                                           ("rl", 576, 4), ("chain", 257, 1), ("chain", 258, 8), ("chain", 321, 2), ("far", 1201, 4)])
def test_units_match_plain_path(kind, n, groups):
    import paper_1807_02431_amd as gpr
    spec = _spec(kind, n)
    print("bonded units", kind, n, groups, flush=True)
    a = gpr.System(spec, path=gpr.PATH_PERSISTENT)
    a.set_launch(0, groups)
    b = gpr.System(spec, path=gpr.PATH_PLAIN)
    rng = np.random.default_rng(n)
    for turn in range(3):
        for k in (1, 20, 11):
            assert np.array_equal(a.advance(k), b.advance(k))
            _same(a, b)
        new = dict(epsilon=spec["epsilon"] * rng.uniform(0.8, 1.2, n), charge=spec["charge"] * rng.uniform(0.8, 1.2, n),
                   torsion_k=spec["torsion_k"] * rng.uniform(0.5, 1.5, len(spec["torsion_k"])))
        for s in (a, b):
            s.set_params(**new)
        if turn == 1:                      # the same terms over other ranges, with the parameters of now
            a.set_launch(0, {1: 2, 2: 4, 4: 8, 8: 1}[groups])
    ea, fa = a.energy_forces()
    eb, fb = b.energy_forces()
    assert np.array_equal(ea, eb) and np.array_equal(fa, fb)
