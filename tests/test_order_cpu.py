"""Host checks of the stage kernels' index arithmetic."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_quotients_and_lds_index(tmp_path):
    """The visiting order's division by multiplication at the edges of its
    range, and the line kernel's LDS index, compiled for the host from the
    kernels' own headers."""
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "div_check")
    cmd = [hipcc, "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(ROOT, "paper_2006_15698_amd", "csrc"), os.path.join(ROOT, "tests", "div_check.cpp"),
           "-o", exe]
    subprocess.run(cmd, check=True, capture_output=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout + out.stderr
    assert "ok" in out.stdout
