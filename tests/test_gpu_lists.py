"""The pair search: a list may hold more pairs than needed but never fewer, so a trajectory does not
depend, to the bit, on how old the lists may get, on the skin or on the masses by which the atoms
move -- nor on the order in which the search took its blocks, tiles and chunks.  Atom counts around
its blocks (8 atoms), tiles (16) and waves, all groupings, mixed and uniform masses, extents beyond
what its products cover (the search then takes distances), and exclusions far apart in index."""
import numpy as np
import pytest

import gpr_synth as G
from test_gpu_small import _same, _spec

pytestmark = pytest.mark.gpu


def _masses(spec, kind):
    n = spec["n_atoms"]
    m = {"as is": spec["mass"], "equal": np.full(n, 14.0), "one light": np.full(n, 16.0),
         "spread": np.geomspace(1.0, 40.0, n)[(7 * np.arange(n)) % n] if n % 7 else spec["mass"]}[kind].copy()
    if kind == "one light":
        m[n // 2] = 1.0
    return dict(spec, mass=m)


@pytest.mark.parametrize("kind,n,groups,masses,shift", [
    ("rl", 161, 1, "as is", 0.0), ("rl", 162, 2, "equal", 0.0), ("rl", 167, 8, "spread", 0.0), ("rl", 168, 1, "one light", 0.0),
    ("far", 169, 8, "as is", 0.0), ("far", 301, 2, "spread", 0.0), ("rl", 433, 4, "spread", 100.0), ("rl", 575, 8, "one light", 300.0),
    ("rl", 1201, 4, "as is", 0.0), ("far", 1203, 8, "as is", 70.0), ("rl", 2432, 8, "as is", 0.0)])
def test_trajectory_does_not_depend_on_the_lists(kind, n, groups, masses, shift):
    import paper_1807_02431_amd as gpr
    spec = _masses(_spec(kind, n), masses)
    if shift:                              # the ligand's restraints are none: it may stand far away
        pos = spec["pos"].copy()
        far = np.arange(n) >= n - 32 if kind == "rl" else np.isin(np.arange(n), (37 * np.arange(n - 32, n)) % n)
        pos[0, far] += shift
        spec["pos"] = pos
    print("lists", kind, n, groups, masses, shift, flush=True)
    base = None
    for path, period, skin in ((gpr.PATH_PERSISTENT, 10, 0.1), (gpr.PATH_PERSISTENT, 1, 0.1), (gpr.PATH_PERSISTENT, 40, 0.02),
                               (gpr.PATH_PERSISTENT, 25, 0.4), (gpr.PATH_PLAIN, 10, 0.1), (gpr.PATH_PLAIN, 3, 0.3)):
        s = gpr.System(dict(spec, nlist_period=period, skin=skin), path=path)
        if path == gpr.PATH_PERSISTENT:
            s.set_launch(0, groups)
        for k in (1, 30, 43):
            s.advance(k)
        if base is None:
            base = s
        else:
            _same(base, s)
    x, v = base.get_state(0)
    assert np.isfinite(x).all() and np.isfinite(v).all()


@pytest.mark.parametrize("n", [1, 2, 7, 8, 9, 15, 16, 17, 63, 64, 65, 130])
def test_forces_do_not_depend_on_the_skin(n):
    """A loose cloud of n atoms (no bonded terms) about the cutoff, on the plain path, near the origin
    and far from it: the same forces with any skin, and those of a sum over all pairs in 64 bits."""
    import paper_1807_02431_amd as gpr
    spec = _spec("chain", 22)
    rng = np.random.default_rng(n)
    grid = np.stack(np.meshgrid(*[np.arange(6)] * 3), -1).reshape(-1, 3)[rng.permutation(216)[:n]]
    spec = dict(spec, n_atoms=n, pos=(0.45 * grid + rng.uniform(-0.08, 0.08, (n, 3))).T.copy(), cutoff=1.0, eps_rf=78.5, nlist_period=10,
                mass=rng.choice([1.0, 12.0, 16.0], n), sigma=rng.uniform(0.2, 0.35, n), epsilon=rng.uniform(0.1, 0.6, n),
                charge=rng.uniform(-0.5, 0.5, n), obs=[],
                state=dict(kind=G.STATE_COM_SPHERE, group=[0], center=[0.0, 0.0, 0.0], radius=1.0))
    for k in list(spec):
        if k.startswith(("bond", "angle", "torsion", "restraint", "pairs14", "exclusions")):
            spec[k] = np.asarray(spec[k])[:0]
    for shift in (0.0, 2000.0):
        pos = spec["pos"] + shift
        out = []
        for skin in (0.02, 0.1, 0.5):
            print("skin", n, shift, skin, flush=True)
            s = gpr.System(dict(spec, pos=pos, skin=skin), path=gpr.PATH_PLAIN)
            out.append(s.energy_forces())
        for e, f in out[1:]:
            assert np.array_equal(e, out[0][0]) and np.array_equal(f, out[0][1])
        x = pos.astype(np.float32).astype(np.float64).T
        d = x[:, None] - x[None]
        r2 = (d ** 2).sum(-1)
        np.fill_diagonal(r2, np.inf)
        ir2 = np.where(r2 < 1.0, 1.0 / r2, 0.0)
        s6 = ((spec["sigma"][:, None] + spec["sigma"]) * 0.5) ** 6 * ir2 ** 3
        e4 = 4.0 * np.sqrt(spec["epsilon"][:, None] * spec["epsilon"])
        qq = 138.935458 * spec["charge"][:, None] * spec["charge"]
        krf = (78.5 - 1.0) / (2.0 * 78.5 + 1.0)
        inside = r2 < 1.0
        w = e4 * (12.0 * s6 * s6 - 6.0 * s6) * ir2 + np.where(inside, qq * (ir2 ** 1.5 - 2.0 * krf), 0.0)
        mag = e4 * (12.0 * s6 * s6 + 6.0 * s6) * ir2 + np.where(inside, abs(qq) * (ir2 ** 1.5 + 2.0 * krf), 0.0)
        ref = (w[..., None] * d).sum(1).T
        scale = (mag[..., None] * np.abs(d)).sum(1).max() + 1.0
        # in units of 2^-24: r^2 3 and its root 2, up to the 14th power, the sum of sigmas 2, to the 12th,
        # and some 15 others, so 100 a pair; n for the sum
        assert np.abs(out[0][1][0] - ref).max() <= (100 + n) * 2.0 ** -24 * scale


@pytest.mark.parametrize("R", [255, 256, 257, 300])
def test_plain_launches_that_fit_the_device_rebuild_jointly(R):
    """Around the number of workgroups up to which a plain launch rebuilds all of its lists as soon as one
    replica has to: the states of the persistent path, with replicas that move very differently."""
    import paper_1807_02431_amd as gpr
    spec = dict(_spec("rl", 161), n_replicas=R, nlist_period=40)
    print("joint rebuilds", R, flush=True)
    a = gpr.System(spec, path=gpr.PATH_PLAIN)
    b = gpr.System(spec, path=gpr.PATH_PERSISTENT)
    for s in (a, b):
        q, v = s.get_state(R - 1)
        s.set_state(R - 1, q, 3.0 * v)         # the fastest comes last
    for k in (1, 25, 40):
        assert np.array_equal(a.advance(k), b.advance(k))
    for r in (0, 1, R // 2, R - 2, R - 1):
        for x, y in zip(a.get_state(r), b.get_state(r)):
            assert np.array_equal(x, y), r
