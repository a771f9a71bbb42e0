"""The gate that orders the resident launches of several contexts, on the CPU: the host
compiler builds tests/host/res_gate_check.cpp, whose threads pass it as the library does."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_launches_of_several_contexts_are_ordered(tmp_path):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("g++ not available")
    csrc = os.path.join(ROOT, "paper_1005_3276_amd", "csrc")
    exe = str(tmp_path / "res_gate_check")
    subprocess.run([cxx, "-O1", "-std=c++17", "-pthread", "-I", csrc,
                    os.path.join(ROOT, "tests", "host", "res_gate_check.cpp"), "-o", exe],
                   check=True, capture_output=True, text=True, timeout=120)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "res_gate ok" in r.stdout
