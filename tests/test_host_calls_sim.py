"""What the host code asks of the device, checked on the CPU over a stand-in for it.

tests/sim/host_calls.cpp defines the HIP calls and the kernel launches that gs_host.cpp
makes and records them, so these cases need no GPU: each is one run of that program.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_26441_amd", "csrc")
HIP_INCLUDE = "/opt/rocm/include"

CASES = ["row_limit", "search_waits_on_the_index_device", "failed_upload_keeps_no_batch",
         "captured_search_has_the_wide_pass", "index_without_room_for_rows",
         "autotune_times_each_launch_once", "listed_queries_fill_the_chip",
         "first_digit_bounds_the_score", "row_terms_at_the_threshold", "update_records"]


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not shutil.which("g++") or not os.path.exists(os.path.join(HIP_INCLUDE, "hip", "hip_runtime.h")):
        pytest.skip("needs g++ and the HIP headers")
    exe = str(tmp_path_factory.mktemp("sim") / "host_calls")
    cmd = ["g++", "-O1", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I", HIP_INCLUDE, "-fsanitize=undefined",
           "-fno-sanitize-recover=all", os.path.join(CSRC, "gs_host.cpp"),
           os.path.join(ROOT, "tests", "sim", "host_calls.cpp"), "-o", exe, "-lpthread"]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-3000:]
    return exe


@pytest.mark.parametrize("case", CASES)
def test_host_calls(program, case):
    r = subprocess.run([program, case], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-1000:] + r.stderr[-2000:]
