"""Host arithmetic of the plans (tables, LDS layouts, dispatch rules) against
what the kernels do with it: tests/host/plan_checks.cpp, built against the
library's own plan source.  No device is used."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1909_13560_amd")


@pytest.fixture(scope="module")
def checks(tmp_path_factory):
    import paper_1909_13560_amd as lib

    lib.load()
    exe = str(tmp_path_factory.mktemp("plan") / "plan_checks")
    hipcc = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("ROCm compilers not available")
    # the kernels' launchers come from the built library
    r = subprocess.run([hipcc, "-x", "hip", "-O1", "-std=c++17", "--offload-arch=gfx950", "-o", exe,
                        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                        os.path.join(ROOT, "tests", "host", "plan_checks.cpp"),
                        "-x", "none", lib.LIB_PATH, f"-Wl,-rpath,{PKG}"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]

    def run(name):
        r = subprocess.run([exe, name], capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stdout + r.stderr

    return run


def test_exact_end_corrections_stay_in_the_window(checks):
    checks("exact_ends")


def test_located_nodes_stay_in_the_window(checks):
    checks("located_windows")


def test_located_windows_do_not_enlarge_the_ring(checks):
    checks("located_ghosts")


def test_shapes_follow_the_measured_times(checks):
    checks("shapes")


def test_fused_or_direct_is_the_faster(checks):
    checks("fused_or_direct")


def test_located_shapes_follow_the_measured_times(checks):
    checks("located_shapes")


def test_exact_kernels_follow_the_measured_times(checks):
    checks("exact_shapes")


def test_plans_copy_their_tables_by_group(checks):
    checks("plan_copies")


def test_the_weights_of_a_plan_sum_to_one(checks):
    checks("weights")
