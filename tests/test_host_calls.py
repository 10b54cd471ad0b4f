"""The library's host code (api.cpp, coeffs.cpp) over a HIP runtime of host
memory that records every launch (tests/host): which kernels a call queues,
what it allocates and what it gives back.  No GPU, no device code."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_22214_amd", "csrc")
HOST = os.path.join(ROOT, "tests", "host")
CLANG = "/opt/rocm/llvm/bin/clang++"

CHECKS = ["restored_velocities", "state_parity", "stepping_allocates_nothing", "other_record_set",
          "batch_autotune_times_its_kernels", "autotune_warms_its_kernels",
          "readback_without_pinned_memory", "readback_from_two_threads", "solid_memory",
          "batch_shares_the_form_of_f", "fused_shapes",
          "mobility_shapes", "batch_runs_share_the_slots",
          "short_calls", "open_faces_wait_for_queued_steps",
          "batch_after_members_stepped"]


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not (os.path.exists(CLANG) or shutil.which("clang++")):
        pytest.skip("no clang++")
    exe = str(tmp_path_factory.mktemp("host") / "host_calls")
    cmd = [CLANG if os.path.exists(CLANG) else "clang++", "-O1", "-g", "-std=c++17", "-pthread",
           "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", f"-I{os.path.join(ROOT, 'include')}", f"-I{CSRC}",
           f"-I{HOST}", os.path.join(CSRC, "coeffs.cpp"), os.path.join(CSRC, "api.cpp"),
           os.path.join(HOST, "fake_hip.cpp"), os.path.join(HOST, "host_calls.cpp"), "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr[-4000:]
    return exe


@pytest.mark.parametrize("check", CHECKS)
def test_host_calls(driver, check):
    run = subprocess.run([driver, check], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout[-2000:] + run.stderr[-2000:]
