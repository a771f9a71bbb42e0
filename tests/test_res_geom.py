"""The resident multi-shift kernel's block decomposition and face addressing on the CPU:
hipcc builds tests/host/res_geom_check.cpp for the host, which checks on a list of lattices
that what every site reads is what its neighbour wrote."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_blocks_tile_and_faces_match(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    csrc = os.path.join(ROOT, "paper_1005_3276_amd", "csrc")
    exe = str(tmp_path / "res_geom_check")
    subprocess.run([hipcc, "-O2", "-std=c++17", "-x", "hip", "--offload-arch=gfx950",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    "-I", csrc, os.path.join(ROOT, "tests", "host", "res_geom_check.cpp"),
                    os.path.join(csrc, "ov_host.cpp"), "-o", exe],
                   check=True, capture_output=True, text=True, timeout=600)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "res_geom ok" in r.stdout
