"""The rotary angles of a run of positions (csrc/hi_rope.h), replayed on the host."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_angles_of_a_run(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path / "rope_check")
    subprocess.run([gxx, "-O2", "-std=gnu++17", "-ffp-contract=off", "-I", os.path.join(ROOT, "paper_2502_12574_amd", "csrc"),
                    os.path.join(ROOT, "tests", "rope_check.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0 and " 0 failures" in r.stdout, r.stdout[-2000:]
