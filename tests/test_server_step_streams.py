"""The server's step when a HIP call of it fails: whatever it had enqueued, on its own stream and
on those forked from it, is waited for before the step returns.  The host code runs on a stand-in
runtime (server_step_streams.cpp), every call of a step failing in turn; no GPU."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ is not installed")
def test_a_failed_step_leaves_no_work_in_flight(tmp_path):
    exe = str(tmp_path / "server_step_streams")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-pthread", "-D__HIP_PLATFORM_AMD__", "-x", "c++", "-w",
                           "-I" + os.path.join(ROCM, "include"), os.path.join(HERE, "server_step_streams.cpp"),
                           "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout.split("calls ")[1].split()[0]) > 20   # the step's calls, all of which failed once
