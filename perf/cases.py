"""Timing cases of the Gen.ParRep library: the calls a program makes, over the sizes it makes them at.

A case is a dict of plain values:
  call      advance   fixed stepping of all replicas on the persistent path (observables, exit checks)
            plain     the same on the plain path, the only one for systems past the persistent kernel's limit
            frames    stepping, then every replica's configuration read back (a trajectory writer)
            walker    transient propagation of the reference walker alone
            dephase   the convergence step: Fleming-Viot branching and Gelman-Rubin at every check
            batch     four systems of different sizes advanced in shared launches
            eval      differentiable energy: forward and backward to positions and parameters
  system    toy (2D double well), chain (vacuum, all pairs) or rl (receptor-ligand, cutoff)
  atoms, replicas, steps   the sizes ("steps" is 0 for eval)

The systems are those of gpr_synth.  A seed sets the noise key (and with it the initial velocities
and every later step), and for eval the positions and parameters; the geometry a system starts from
depends on its size alone.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import gpr_synth as G
import paper_1807_02431_amd as gpr
from paper_1807_02431_amd.autograd import EnergyModel

COULOMB_F = 138.935458          # kJ mol^-1 nm e^-2
LIGAND = 32                     # ligand atoms of every receptor-ligand system
RADIUS = {300: 2.2, 1200: 3.2, 2432: 4.0, 4600: 5.0, 5200: 5.2}     # sphere of the named sizes, nm
# floating-point operations (a fused multiply-add counts two) per unit of work
FLOP_PAIR, FLOP_PAIR_GRAD, FLOP_ATOM = 40, 30, 20
FLOP_BOND, FLOP_ANGLE, FLOP_TORSION, FLOP_RESTRAINT, FLOP_PAIR14 = 25, 60, 110, 12, 45


def listed():
    def c(name, call, system, atoms, replicas, steps):
        return dict(name=name, call=call, system=system, atoms=atoms, replicas=replicas, steps=steps)
    return [
        # the smallest call there is: one particle, eight walkers, one check period; all latency
        c("toy_check", "advance", "toy", 1, 8, 10),
        # the alanine-dipeptide-sized chain: the reference walker's residence time (one replica) ...
        c("chain22_walker", "walker", "chain", 22, 256, 500),
        # ... and its convergence step with a check every 250 steps
        c("chain22_dephase", "dephase", "chain", 22, 256, 1000),
        # force-field fitting on the chain: many small configurations per evaluation
        c("chain22_eval", "eval", "chain", 22, 256, 0),
        # a small receptor-ligand system whose replicas are all written out after a short run
        c("rl300_frames", "frames", "rl", 300, 24, 50),
        # more replicas than the device holds at once, at a middle size
        c("rl1200_steps", "advance", "rl", 1200, 192, 50),
        # the benchmark workload in short calls, where a launch's start and end count ...
        c("rl2432_short", "advance", "rl", 2432, 64, 20),
        # ... and in one whole check period with its check
        c("rl2432_check", "advance", "rl", 2432, 64, 1000),
        # the reference walker of that system alone, one check period
        c("rl2432_walker", "walker", "rl", 2432, 64, 1000),
        # energy, forces and parameter gradient of all its replicas
        c("rl2432_eval", "eval", "rl", 2432, 64, 0),
        # a system past the persistent kernel's limit, on the plain path
        c("rl5200_plain", "plain", "rl", 5200, 12, 20),
        # the four sizes of the uneven mix in shared launches
        c("uneven_batch", "batch", "mix", 0, 48, 50),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    call = rng.choice(["advance", "advance", "advance", "plain", "frames", "walker", "dephase", "batch", "eval", "eval"])
    if call == "batch":
        return dict(call=call, system="mix", atoms=0, replicas=_log(rng, 3, 96), steps=_log(rng, 5, 100))
    system = rng.choice(["chain", "rl", "rl", "rl"] if call != "advance" else ["toy", "chain", "rl", "rl", "rl"])
    if system == "toy":
        return dict(call=call, system=system, atoms=1, replicas=_log(rng, 2, 512), steps=_log(rng, 5, 500))
    if system == "chain":
        atoms, replicas = _log(rng, 14, 60), _log(rng, 2, 512)
    else:
        atoms = _log(rng, 60, 5200 if call in ("plain", "eval") else 4600)
        replicas = _log(rng, 2, max(2, min(256, 64 * 2432 // atoms)))
    if call == "frames":
        replicas = min(replicas, 32)
    if call == "eval":
        return dict(call=call, system=system, atoms=atoms, replicas=replicas, steps=0)
    # no dearer than a whole check period of the 2,432-atom system: 1,000 steps of 64 replicas
    share = max(atoms * replicas / (2432 * 64), atoms / 2432, 0.25) * (4 if call == "plain" else 1)
    steps = _log(rng, 5, max(5, int(min(1000, 800 / share))))
    return dict(call=call, system=system, atoms=atoms, replicas=replicas, steps=steps)


# ------------------------------------------------------------------ inputs
def _radius(atoms):
    return RADIUS.get(atoms) or max(1.7, 4.4 * ((atoms - LIGAND) / 2400.0) ** (1.0 / 3.0))


def _spec(system, atoms, replicas, key, t_check=None):
    if system == "toy":
        s = G.toy2d(n_replicas=replicas)
    elif system == "chain":
        s = G.chain(n_atoms=atoms, n_replicas=replicas)
    else:
        s = G.receptor_ligand(n_receptor=atoms - LIGAND, radius=_radius(atoms), n_replicas=replicas)
    s = G.round_to_f32(s)
    s["seed"] = (int(key) * 0x9E3779B97F4A7C15 + 12345) % (1 << 63)
    if t_check:
        s["t_check_dephase"] = t_check
    return s


def _specs(case, seed):
    """Descriptors of the case's systems (one, or the four of the uneven mix)."""
    if case["call"] == "batch":
        R = case["replicas"]
        return [_spec("chain", 22, R, 4 * seed)] + [_spec("rl", n, R, 4 * seed + 1 + k) for k, n in enumerate((300, 1200, 2432))]
    # the walker is tested at the end of its residence time
    return [_spec(case["system"], case["atoms"], case["replicas"], seed, case["steps"] if case["call"] == "walker" else None)]


def _eval_inputs(spec, seed, device):
    """Positions around the start configuration and parameters around the force field's, from the seed."""
    g = np.random.default_rng(seed)
    R, n = spec["n_replicas"], spec["n_atoms"]
    x = (spec["pos"][None] + g.normal(0.0, 0.004, (R, 3, n))).astype(np.float32)
    p = [np.asarray(spec[k], np.float64) * (1.0 + 0.02 * g.uniform(-1.0, 1.0, len(spec[k])))
         for k in ("epsilon", "sigma", "charge", "torsion_k")]
    return torch.tensor(x, device=device), [torch.tensor(a, device=device) for a in p]


def prepare(case, seed):
    specs = _specs(case, seed)
    st = dict(case=case)
    if case["call"] == "eval":
        st["model"] = EnergyModel(specs[0])
        x, p = _eval_inputs(specs[0], seed, "cuda")
        st["leaves"] = [t.requires_grad_() for t in [x] + p]
        return st
    path = gpr.PATH_PLAIN if case["call"] == "plain" else gpr.PATH_PERSISTENT
    st["systems"] = [gpr.System(s, path=path, stream=torch.cuda.current_stream()) for s in specs]
    return st


# ------------------------------------------------------------------ one pass
def _sums_and_walker(s):
    n, S1, S2, shift = s.accumulators()
    q, v = s.get_state(0)
    return dict(samples=n, S1=S1, S2=S2, shift=shift, q=q, v=v)


def run(st):
    c = st["case"]
    call, k = c["call"], c["steps"]
    if call == "eval":
        U = st["model"](*st["leaves"])
        return dict(U=U.detach(), grads=list(torch.autograd.grad(U.sum(), st["leaves"])))
    s = st["systems"][0]
    if call in ("advance", "plain"):
        return dict(first_exit=s.advance(k), **_sums_and_walker(s))
    if call == "frames":
        fec = s.advance(k)
        frames = [s.get_state(r) for r in range(s.R)]
        return dict(first_exit=fec, q=np.stack([f[0] for f in frames]), v=np.stack([f[1] for f in frames]))
    if call == "walker":
        rc, ev = s.decorrelate(k, max_steps=k)
        q, v = s.get_state(0)
        return dict(status=rc, event=ev, q=q, v=v)
    if call == "dephase":
        rc, o = s.dephase(max_steps=k)
        return dict(status=rc, result=o, **_sums_and_walker(s))
    fec = gpr.batch_advance(st["systems"], k)
    return [dict(first_exit=f, **_sums_and_walker(x)) for f, x in zip(fec, st["systems"])]


# ------------------------------------------------------------------ work a pass cannot do without
@functools.lru_cache(maxsize=64)
def _pairs(system, atoms):
    """In-cutoff pairs of one replica that are neither excluded nor 1-4 (more than three bonds apart)."""
    if system == "toy":
        return 0
    if system == "chain":
        return (atoms - 3) * (atoms - 4) // 2
    s = _spec("rl", atoms, 2, 0)
    x, tot = s["pos"].T, 0
    for i in range(atoms):
        d = x[i + 4:] - x[i]
        tot += int(((d * d).sum(1) < s["cutoff"] ** 2).sum())
    return tot


def work(case):
    b = f = 0
    sizes = [("chain", 22), ("rl", 300), ("rl", 1200), ("rl", 2432)] if case["call"] == "batch" else [(case["system"], case["atoms"])]
    for system, n in sizes:
        R, k = (1 if case["call"] == "walker" else case["replicas"]), max(1, case["steps"])
        mol = system != "toy"
        terms = n * (FLOP_BOND + FLOP_ANGLE + FLOP_TORSION + FLOP_PAIR14 + (FLOP_RESTRAINT if system == "rl" else 0)) if mol else 10
        topo = n * (16 + 4 + (16 + 24 + 32 + 24 + 20 if mol else 0))      # parameters and terms, once
        if case["call"] == "eval":
            f += R * (_pairs(system, n) * (FLOP_PAIR + FLOP_PAIR_GRAD) + terms)
            b += topo + R * (n * 24 + 8) + n * 32
        else:
            f += R * k * (_pairs(system, n) * FLOP_PAIR + terms + n * FLOP_ATOM)
            b += topo + R * n * 48                                         # x and v, in and out
    return dict(bytes=b, flops=f)


# ------------------------------------------------------------------ the same in 64 bits
def _philox(ctr, key):
    """Philox4x32-10 (Salmon et al., SC'11) on uint64 arrays holding 32-bit words."""
    m, (k0, k1), (a, b, c, d) = np.uint64(0xFFFFFFFF), key, ctr
    for _ in range(10):
        p0, p1 = a * np.uint64(0xD2511F53), c * np.uint64(0xCD9E8D57)
        a, b, c, d = (p1 >> np.uint64(32)) ^ b ^ np.uint64(k0), p1 & m, (p0 >> np.uint64(32)) ^ d ^ np.uint64(k1), p0 & m
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return a, b, c, d


def _gauss(seed, n, replicas, step, stream):
    """[replicas][3][n] Gaussians of the library's noise convention (gpr.h)."""
    a = np.arange(n, dtype=np.uint64)[None, :]
    r = np.arange(replicas, dtype=np.uint64)[:, None]
    o = np.zeros((replicas, n), np.uint64)
    w = _philox((a + o, o + np.uint64(step), r + o, o + np.uint64(stream << 24)), (seed & 0xFFFFFFFF, seed >> 32))
    u = [(2.0 * (x >> np.uint64(9)).astype(np.float64) + 1.0) * 2.0 ** -24 for x in w]
    ra, rb = np.sqrt(-2.0 * np.log(u[0])), np.sqrt(-2.0 * np.log(u[2]))
    return np.stack([ra * np.cos(2 * np.pi * u[1]), ra * np.sin(2 * np.pi * u[1]), rb * np.cos(2 * np.pi * u[3])], 1)


class _Field:
    """The potential energy of gpr.h in float64, for torch.autograd."""

    def __init__(self, spec, device):
        self.s, self.n, self.dev = spec, spec["n_atoms"], device
        self.toy = spec["kind"] == G.TOY2D
        if self.toy:
            return
        t = lambda a: torch.tensor(np.asarray(a), device=device)  # noqa: E731
        self.par = [t(np.asarray(spec[k], np.float64)) for k in ("epsilon", "sigma", "charge", "torsion_k")]
        self.ix = {k: t(np.asarray(spec[k], np.int64)) for k in ("bonds", "angles", "torsions", "restraints", "pairs14")}
        self.c = {k: t(np.asarray(spec[k], np.float64)) for k in
                  ("bond_r0", "bond_k", "angle_theta0", "angle_k", "torsion_n", "torsion_phi0", "restraint_ref", "restraint_k")}
        keep = np.triu(np.ones((self.n, self.n), bool), 1)
        for i, j in np.concatenate([spec["exclusions"], spec["pairs14"]]):
            keep[min(i, j), max(i, j)] = False
        self.keep = t(keep)

    def __call__(self, x, par=None):
        """x [3][n] -> U (one replica)"""
        if self.toy:
            return (x[0, 0] ** 2 - 1) ** 2 + 2 * x[1, 0] ** 2
        eps, sig, q, tk = par or self.par
        s, c, X = self.s, self.c, x.T
        d = X[self.ix["bonds"][:, 1]] - X[self.ix["bonds"][:, 0]]
        U = (0.5 * c["bond_k"] * (d.norm(dim=1) - c["bond_r0"]) ** 2).sum()
        i, j, k = self.ix["angles"].T
        u, w = X[i] - X[j], X[k] - X[j]
        U = U + (0.5 * c["angle_k"] * (torch.atan2(torch.linalg.cross(u, w).norm(dim=1), (u * w).sum(1)) - c["angle_theta0"]) ** 2).sum()
        i, j, k, m = self.ix["torsions"].T
        b1, b2, b3 = X[j] - X[i], X[k] - X[j], X[m] - X[k]
        n1, n2 = torch.linalg.cross(b1, b2), torch.linalg.cross(b2, b3)
        phi = torch.atan2(b2.norm(dim=1) * (b1 * n2).sum(1), (n1 * n2).sum(1))
        U = U + (tk * (1 + torch.cos(c["torsion_n"] * phi - c["torsion_phi0"]))).sum()
        if len(self.ix["restraints"]):
            U = U + (0.5 * c["restraint_k"] * ((X[self.ix["restraints"]] - c["restraint_ref"]) ** 2).sum(1)).sum()
        i, j = self.ix["pairs14"].T
        U = U + s["scale14"] * self._pair(X[i], X[j], eps[i], eps[j], sig[i], sig[j], q[i], q[j], 0.0, 0.0).sum()
        with torch.no_grad():
            near = self.keep
            if s["cutoff"] > 0:
                r2 = sum((x[a][:, None] - x[a][None, :]) ** 2 for a in range(3))
                near = near & (r2 < s["cutoff"] ** 2)
            i, j = near.nonzero(as_tuple=True)
        rc = s["cutoff"]
        krf = (s["eps_rf"] - 1) / ((2 * s["eps_rf"] + 1) * rc ** 3) if rc > 0 else 0.0
        crf = 1 / rc + krf * rc * rc if rc > 0 else 0.0
        return U + self._pair(X[i], X[j], eps[i], eps[j], sig[i], sig[j], q[i], q[j], krf, crf).sum()

    @staticmethod
    def _pair(a, b, ea, eb, sa, sb, qa, qb, krf, crf):
        r2 = ((a - b) ** 2).sum(1)
        r = torch.sqrt(r2)
        s6 = (0.5 * (sa + sb) / r) ** 6
        return 4 * torch.sqrt(ea * eb) * (s6 * s6 - s6) + COULOMB_F * qa * qb * (1 / r + krf * r2 - crf)


def _follow(spec, replicas, steps, device):
    """(q, v) of replicas [0, replicas) after `steps` BAOAB steps from the start, [replicas][3][n]."""
    F, n, seed = _Field(spec, device), spec["n_atoms"], spec["seed"]
    m = torch.tensor(np.asarray(spec["mass"], np.float64), device=device)
    dt, kT = spec["dt"], spec["kT"]
    c1 = math.exp(-spec["gamma"] * dt)
    flat = torch.tensor([1.0, 1.0, 0.0 if F.toy else 1.0], dtype=torch.float64, device=device)[:, None]
    g = lambda step, stream, R: torch.tensor(_gauss(seed, n, R, step, stream), device=device) * flat  # noqa: E731
    x = torch.tensor(spec["pos"], device=device).repeat(replicas, 1, 1)
    v = (torch.sqrt(kT / m) * g(0, 1, 1)).repeat(replicas, 1, 1)

    def forces(x):
        y = x.detach().requires_grad_()
        return torch.stack([-torch.autograd.grad(F(y[r]), y)[0][r] for r in range(replicas)])

    f = forces(x)
    for s in range(steps):
        x = x + 0.5 * dt * (v + 0.5 * dt * f / m)
        v = c1 * (v + 0.5 * dt * f / m) + torch.sqrt((1 - c1 * c1) * kT / m) * g(s, 0, replicas)
        x = x + 0.5 * dt * v
        f = forces(x)
        v = v + 0.5 * dt * f / m
    return x.cpu().numpy(), v.cpu().numpy()


def exact(case, seed):
    call, k, R = case["call"], case["steps"], case["replicas"]
    device = "cuda" if torch.cuda.is_available() else "cpu"
    if call == "batch":
        return None
    spec = _specs(case, seed)[0]
    if call == "eval":
        F = _Field(spec, device)
        x, p = _eval_inputs(spec, seed, device)
        p = [t.requires_grad_() for t in p]
        U, gx, gp = [], [], [torch.zeros_like(t) for t in p]
        for r in range(R):
            y = x[r].double().requires_grad_()
            u = F(y, p)
            g = torch.autograd.grad(u, [y] + p)
            U.append(u.detach())
            gx.append(g[0])
            gp = [a + b for a, b in zip(gp, g[1:])]
        return dict(U=torch.stack(U), grads=[torch.stack(gx)] + gp)
    # trajectories diverge from their 64-bit counterpart exponentially: short ones only
    many = R if call == "frames" else 1
    if k > 100 or k * many > 1500 or call == "dephase":
        return None
    q, v = _follow(spec, many, k, device)
    if call == "frames":
        return dict(first_exit=None, q=q, v=v)
    q, v = q[0], v[0]
    if call == "walker":
        return dict(status=None, event=None, q=q, v=v)
    return dict(first_exit=None, samples=None, S1=None, S2=None, shift=None, q=q, v=v)
