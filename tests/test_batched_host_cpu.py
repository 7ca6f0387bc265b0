"""The batched path's host code on the CPU (paper_2207_00257_amd/csrc/
nrm_batched_api.cpp) with a HIP runtime over host memory in place of the GPU's
(tests/cpu/batched_host_test.cpp): the launches' shapes over
all row counts, the row tables of captured calls, the work lists after
a failed launch, the workspace's arrays, the summation tree's height.
Built with g++ only, under AddressSanitizer and UndefinedBehaviorSanitizer."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "cpu", "batched_host_test.cpp")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("batched_host") / "driver")
    cmd = ["g++", "-O1", "-g", "-std=c++17", "-pthread", "-Wall", "-D__HIP_PLATFORM_AMD__",
           "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
           "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2207_00257_amd", "csrc"),
           "-isystem", os.path.join(ROCM, "include"), SRC, "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    return exe


@pytest.mark.parametrize("case", ["rows_grid", "captured_tables", "failed_launch", "workspace_layout", "tree_height",
                                  "apart_rule", "cuts_without_resident_rows", "cuts_of_wavefront_rows",
                                  "cuts_of_one_segment_rows"])
def test_batched_host(driver, case):
    r = subprocess.run([driver, case], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
