"""The host runtime built with g++ against a CPU stand-in of the HIP runtime
(tests/host_harness) whose launchers record what they are given.  No GPU.

arrays: a blocking solve reads device inputs and writes device results where
they are only if the device holds the whole array; any other one is staged.
budget: requests that run in slices of 64 paths claim memory for the slices'
records only beside all else that is in use or waits, so they run together
wherever whole chunks would, within the budget.
boxes: a forced LDS solve runs the LDS kernel for every subdomain that fits it.
jobs: the jobs of windowed launches hold every item once, in as many as the
workgroups need.
slices: no slices where many of their lanes would have no path.
fp64: FP64 requests are charged for the partial sums that they allocate, and
fit every budget that items of 256 paths fitted."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HARNESS = os.path.join(ROOT, "tests", "host_harness")
CSRC = os.path.join(ROOT, "paper_1504_00084_amd", "csrc")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("g++ not available")
    out = os.path.join(str(tmp_path_factory.mktemp("calls")), "calls")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-I" + HARNESS, "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
           os.path.join(CSRC, "runtime.cpp"), os.path.join(CSRC, "mesh_step.cpp"), os.path.join(HARNESS, "calls.cpp"),
           "-o", out, "-lpthread"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]
    return out


@pytest.mark.parametrize("scenario", ["arrays", "budget", "boxes", "jobs", "slices", "fp64"])
def test_calls(exe, scenario):
    res = subprocess.run([exe, scenario], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0 and "all checks passed" in res.stdout, (res.stdout + res.stderr)[-4000:]
