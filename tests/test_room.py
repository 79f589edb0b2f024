"""Room for launches whose workgroups wait for one another (host code, no GPU): what is taken at a time never
exceeds the device, launches on one stream share, nobody overtakes who waits, and threads that take and
give at random all come to their end."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1807_02431_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_room_never_exceeds_the_device(tmp_path):
    exe = str(tmp_path / "room")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-pthread", "-I" + CSRC, os.path.join(HERE, "room_check.cpp"), "-o", exe])
    p = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert p.returncode == 0 and p.stdout.strip() == "ok", p.stdout
