"""Atom ranges of the workgroups of a replica (host code, no GPU): they cover the replica in order, start
at multiples of 16 and are never empty, for tiny replicas, more workgroups than blocks of 16 atoms
and strongly uneven work; where the boundaries that the work alone asks for leave no range empty, they are those."""
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1807_02431_amd", "csrc")


def _works():
    rng = np.random.default_rng(3)
    out = []
    for n in (1, 2, 14, 16, 17, 22, 31, 32, 33, 60, 63, 64, 100, 127, 129, 161, 300, 511, 1024, 1025, 2432):
        ramp = 72.0 + np.linspace(0, 400, n)
        dense = np.full(n, 72.0)
        dense[: n // 6 + 1] = 900.0        # a packed core on a loose chain
        spike = np.full(n, 72.0)
        spike[n // 2] = 1e5
        out += [np.ones(n), ramp, dense, dense[::-1], spike, 72.0 + 300.0 * rng.random(n)]
    return out


def _by_work(w, G):
    """Boundaries where the running sum crosses g / G, at the nearer multiple of 16."""
    n, cum, b = len(w), np.concatenate([[0.0], np.cumsum(w)]), [0]
    for g in range(1, G):
        t = cum[n] * g / G
        lo = int(np.searchsorted(cum, t)) // 16 * 16
        hi = min(n, lo + 16)
        b.append(min(n, max(lo if t - cum[lo] <= cum[hi] - t else hi, b[-1])))
    return b + [n]


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_no_range_is_empty(tmp_path):
    exe = str(tmp_path / "ranges")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I" + CSRC, os.path.join(HERE, "atom_ranges_check.cpp"), "-o", exe])
    ask = [(w, G) for w in _works() for G in (1, 2, 4, 8, 16, 32)]
    text = "".join("%d %d %s\n" % (len(w), G, " ".join(repr(float(x)) for x in w)) for w, G in ask)
    lines = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
    assert len(lines) == len(ask)
    empty_by_work = 0
    for (w, G), line in zip(ask, lines):
        n, (g, lmax, *bnd) = len(w), [int(x) for x in line.split()]
        blocks = (n + 15) // 16
        assert g == max(k for k in (1, 2, 4, 8, 16, 32) if k <= min(G, blocks)), (n, G)
        assert bnd[0] == 0 and bnd[-1] == n and len(bnd) == g + 1
        size = np.diff(bnd)
        assert (size > 0).all() and all(b % 16 == 0 for b in bnd[:-1]), (n, G, bnd)
        assert g == 1 or (lmax % 16 == 0 and lmax - 16 < size.max() <= lmax)
        plain = _by_work(w, G)
        if (np.diff(plain) > 0).all():
            assert bnd == plain, (n, G)
        else:
            empty_by_work += 1
    assert empty_by_work > 100              # the cases this is about are among them
