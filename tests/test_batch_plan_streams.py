"""The side streams of a batch plan.  A search in block form runs in a kernel of its size and
symmetry, so small batches that were one kernel in tiles are several; for short searches they run
one after another on the caller's stream, since making side streams and passing events would take
longer than they save.  When a call of a run fails, the lanes it had started are joined to the
caller's stream all the same.  The host code runs on a stand-in runtime (standin_hip.h); no GPU."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ is not installed")
def test_side_streams_of_short_and_long_plans(tmp_path):
    exe = str(tmp_path / "batch_plan_streams")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-pthread", "-D__HIP_PLATFORM_AMD__", "-x", "c++", "-w",
                           "-I" + os.path.join(ROCM, "include"), os.path.join(HERE, "batch_plan_streams.cpp"),
                           "-o", exe])
    env = {k: v for k, v in os.environ.items() if k not in ("QAP_BATCH_LANES", "GPU_MAX_HW_QUEUES")}
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60, env=env)
    assert r.returncode == 0, r.stdout
    out = [int(x) for x in r.stdout.split()]
    assert out[:9] == [0, 0, 0, 1, 0, 0, 2, 1, 1], r.stdout
    assert out[9] == 0 and out[10] > 10, (r.stdout, r.stderr)
