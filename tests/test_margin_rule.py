"""Which atoms get half the skin as their pair-list margin (host code, no GPU): those of less than four times the
lightest's mass, and no others; the others' share follows the lightest of them."""
import math
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1807_02431_amd", "csrc")

MASSES = [[1.0], [12.0, 12.0], [1.0, 12.0, 14.0, 16.0], [1.0, 2.5, 16.0], [1.0, 1.9, 2.0, 2.1, 3.999, 4.0, 4.001],
          [1.0, 3.9], [2.0, 7.9, 8.0], [1.0, 1e6], [12.011, 1.008, 15.999, 4.1], [1e-30, 3e-30, 5e-30]]


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_light_atoms_are_those_below_four_times_the_lightest(tmp_path):
    exe = str(tmp_path / "margins")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I" + CSRC, os.path.join(HERE, "margin_rule_check.cpp"), "-o", exe])
    text = "".join("%d %s\n" % (len(m), " ".join(map(repr, m))) for m in MASSES)
    lines = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
    assert len(lines) == len(MASSES)
    for m, line in zip(MASSES, lines):
        heavy, *light = line.split()
        low = min(m)
        assert [int(x) for x in light] == [int(x < 4.0 * low) for x in m], m
        over = [x for x in m if x >= 4.0 * low]
        assert float(heavy) == pytest.approx(min(1.0, 1.35 * math.sqrt(low / min(over))) if over else 1.0, rel=1e-12)
