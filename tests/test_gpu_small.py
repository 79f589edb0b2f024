"""The kernel of small replicas (one workgroup each, at most 160 atoms with a cutoff, 256 without, no pair lists) against the
plain path, bit for bit: positions, velocities, accumulators and first exit checks, at the edges of
its units (64 bonded terms, 16 atoms of a pair task, 64 Gaussians), over block sizes from one wave
to sixteen, with and without a cutoff, and with the path changed under way (the launch keeps no
list, so the next kernel that needs one has to build it)."""
import sys

import numpy as np
import pytest

import gpr_synth as G

pytestmark = pytest.mark.gpu


def _spec(kind, n):
    if kind == "toy":
        return G.toy2d(n_replicas=5)
    if kind == "chain":
        return G.chain(n_atoms=n, n_replicas=3, t_check=50)
    s = G.receptor_ligand(n_receptor=n - 32, radius=max(1.7, 4.4 * ((n - 32) / 2400.0) ** (1 / 3)), n_replicas=3, t_gr=7, t_check=20)
    if kind == "far":                     # atom k becomes 37 k mod n: bonded neighbours far apart in index
        to = (37 * np.arange(n)) % n
        assert len(set(to)) == n
        inv = np.argsort(to)
        for k in ("mass", "sigma", "epsilon", "charge"):
            s[k] = s[k][inv]
        s["pos"] = s["pos"][:, inv]
        for k in ("bonds", "angles", "torsions", "restraints", "pairs14", "exclusions"):
            s[k] = to[s[k]].astype(np.int32)
        s["state"] = dict(s["state"], group=to[s["state"]["group"]].astype(np.int32))
        s["obs"] = [dict(o, **{g: to[o[g]].astype(np.int32) for g in ("group_a", "group_b") if o.get(g) is not None}) for o in s["obs"]]
    return s


def _same(a, b):
    for r in range(a.R):
        for x, y in zip(a.get_state(r), b.get_state(r)):
            assert np.array_equal(x, y), r
    for x, y in zip(a.accumulators(), b.accumulators()):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("kind,n,bt", [("toy", 1, 64), ("toy", 1, 256), ("chain", 14, 64), ("chain", 22, 128), ("chain", 22, 448),
                                       ("chain", 63, 320), ("chain", 64, 64), ("chain", 65, 1024), ("chain", 67, 704),
                                       ("chain", 256, 1024), ("rl", 80, 512), ("rl", 128, 1024), ("rl", 159, 192),
                                       ("rl", 160, 1024), ("far", 100, 1024), ("rl", 161, 1024), ("chain", 257, 1024)])
def test_small_kernel_matches_plain_path(kind, n, bt):
    import paper_1807_02431_amd as gpr
    spec = _spec(kind, n)
    print("small kernel", kind, n, bt, flush=True)
    sys.stdout.flush()
    a = gpr.System(spec, path=gpr.PATH_PERSISTENT)
    a.set_launch(bt, 1)
    b = gpr.System(spec, path=gpr.PATH_PLAIN)
    for k in (1, 3, 40, 17, 60):
        assert np.array_equal(a.advance(k), b.advance(k))
        _same(a, b)
    a.set_path(gpr.PATH_PLAIN)            # plain steps straight after a launch that kept no list
    assert np.array_equal(a.advance(13), b.advance(13))
    a.set_path(gpr.PATH_PERSISTENT)
    a.set_launch(0, 2)                    # and the general kernel after those, then after small launches
    assert np.array_equal(a.advance(12), b.advance(12))
    a.set_launch(0, 1)
    assert np.array_equal(a.advance(5), b.advance(5))
    a.set_launch(0, 2)
    assert np.array_equal(a.advance(9), b.advance(9))
    _same(a, b)
    ea, fa = a.energy_forces()
    eb, fb = b.energy_forces()
    assert np.array_equal(ea, eb) and np.array_equal(fa, fb)


@pytest.mark.parametrize("kind,n,R", [("rl", 140, 3), ("rl", 300, 3), ("rl", 300, 100), ("rl", 600, 40), ("chain", 22, 300)])
def test_launch_shape_by_replica_count(kind, n, R):
    """The shape a launch takes by itself (workgroups per replica and threads by the number of
    replicas stepped, one for the walker's steps) against fixed shapes: the same events and states."""
    import paper_1807_02431_amd as gpr
    spec = dict(_spec(kind, n), n_replicas=R, t_check_dephase=20)
    print("launch shape", kind, n, R, flush=True)
    a = gpr.System(spec, path=gpr.PATH_PERSISTENT)
    b = gpr.System(spec, path=gpr.PATH_PERSISTENT)
    b.set_launch(256, 2)
    for k in (0, 1):
        assert a.decorrelate(40, max_steps=40) == b.decorrelate(40, max_steps=40)
        assert np.array_equal(a.advance(25), b.advance(25))
    for r in (0, 1, R // 2, R - 1):
        for x, y in zip(a.get_state(r), b.get_state(r)):
            assert np.array_equal(x, y), r
