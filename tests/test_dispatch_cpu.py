"""Host checks of the rules by which a launch's order and kernel are chosen,
compiled from the library's own headers and sources."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _run(tmp_path, name, libs=()):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / name)
    cmd = [hipcc, "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(ROOT, "paper_2006_15698_amd", "csrc"), os.path.join(ROOT, "tests", name + ".cpp"),
           "-o", exe, *libs]
    subprocess.run(cmd, check=True, capture_output=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout + out.stderr
    assert "ok" in out.stdout


def test_blocks_shared_by_the_xcds(tmp_path):
    """Meshes whose planes hold few blocks (long in z) do not scatter
    neighbouring blocks over the XCDs, and every block is still visited once."""
    _run(tmp_path, "order_rules_check")


def test_line_or_node_kernels(tmp_path):
    """Small launches, short rows and nearly empty last rounds go to the
    kernels with a thread per node."""
    _run(tmp_path, "line_rules_check")
