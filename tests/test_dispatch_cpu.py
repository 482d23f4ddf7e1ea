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


def test_pencil_depth_option_round_trips():
    """DG_OPT_PENCIL_Z reads as the depth that the stages use; writing back
    what was read keeps it, and DG_OPT_PENCIL_Z_AUTO goes back to automatic."""
    from paper_2006_15698_amd import dg
    for n, p, prec, depth in ((48, 4, dg.DG_FP64, 1), (48, 4, dg.DG_FP32_MFMA, 4), (32, 3, dg.DG_FP64, 8),
                              (96, 0, dg.DG_FP64, 8), (160, 0, dg.DG_FP64, 4)):
        ctx = dg.dg_create(n, n, n, p, 1.4)
        try:
            dg.dg_set_precision(ctx, prec)
            read = lambda: (dg.dg_get_option(ctx, dg.DG_OPT_PENCIL_Z), dg.dg_get_option(ctx, dg.DG_OPT_PENCIL_Z_AUTO))
            assert read() == (depth, 1)
            before = {k: dg.dg_get_option(ctx, k) for k in dg.OPTION_NAMES}
            for k, v in before.items():
                dg.dg_set_option(ctx, k, v)
            assert {k: dg.dg_get_option(ctx, k) for k in dg.OPTION_NAMES} == before
            dg.dg_set_option(ctx, dg.DG_OPT_PENCIL_Z, depth)
            assert read() == (depth, 0)
            dg.dg_set_option(ctx, dg.DG_OPT_PENCIL_Z, 3)
            assert read() == (3, 0)
            dg.dg_set_option(ctx, dg.DG_OPT_PENCIL_Z_AUTO, 1)
            assert read() == (depth, 1)
            dg.dg_set_option(ctx, dg.DG_OPT_XCD_REMAP, 0)
            assert read() == (8, 1)
        finally:
            dg.dg_destroy(ctx)


def test_batch_window_option():
    """Every deal of a batch's items can be had and read back."""
    from paper_2006_15698_amd import dg
    b = dg.dg_batch_create([(4, 4, 4)], [3], [(1.0, 1.0, 1.0)])
    try:
        read = lambda: (dg.dg_batch_get_option(b, dg.DG_OPT_XCD_REMAP), dg.dg_batch_get_option(b, dg.DG_OPT_XCD_WINDOW))
        assert read() == (0, 1)
        for xcd, window in ((0, 0), (1, 0), (1, 1), (0, 1)):
            dg.dg_batch_set_option(b, dg.DG_OPT_XCD_REMAP, xcd)
            dg.dg_batch_set_option(b, dg.DG_OPT_XCD_WINDOW, window)
            assert read() == (xcd, window)
    finally:
        dg.dg_batch_destroy(b)
    ctx = dg.dg_create(4, 3, 2, 3, 1.4)
    try:
        with pytest.raises(dg.DGError):   # not an option of a single mesh
            dg.dg_set_option(ctx, dg.DG_OPT_XCD_WINDOW, 0)
    finally:
        dg.dg_destroy(ctx)


def test_variable_degree_lists_beyond_the_cache(tmp_path):
    """The element lists of meshes whose arrays exceed the last-level cache
    are partitions by (degree, size), wide, thin and flat meshes, refined and
    not."""
    from paper_2006_15698_amd import dg
    libdir = os.path.dirname(dg.LIB_PATH)
    _run(tmp_path, "varp_list_check", ("-L", libdir, "-ldg", f"-Wl,-rpath,{libdir}"))
