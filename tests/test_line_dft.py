"""The LDS line transforms of the momentum-space kernels (any even length up to 64), run on
the CPU: hipcc builds tests/host/line_dft_check.cpp for the host."""
import os
import subprocess

from test_line_fft import ROOT, _hipcc


def test_line_dft_matches_direct_dft(tmp_path):
    exe = str(tmp_path / "line_dft_check")
    subprocess.run([_hipcc(), "-O2", "-std=c++17", "-x", "hip", "--offload-arch=gfx950",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    "-I", os.path.join(ROOT, "paper_1005_3276_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "line_dft_check.cpp"), "-o", exe],
                   check=True, capture_output=True, text=True, timeout=600)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "line_dft ok" in r.stdout
