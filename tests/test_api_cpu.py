"""The C ABI's host side without a GPU: paper_2609_33814_amd/csrc/bdrs_api.hip
compiled by the host compiler against a simulated runtime (tests/api_driver.cpp),
which sees in what order a call launches, waits and fails."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_33814_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None or not os.path.exists(os.path.join(ROCM, "include", "hip", "hip_runtime.h")):
        pytest.skip("g++ or the HIP headers are not available")
    exe = str(tmp_path_factory.mktemp("api") / "api_driver")
    # what hipcc's own headers would define
    hip = ["-D__HIP_PLATFORM_AMD__", "-D__align__(n)=__attribute__((aligned(n)))", "-DHIP_SYMBOL(x)=x"]
    cmd = [cxx, "-std=c++17", "-O1", *hip, "-I", CSRC, "-I", os.path.join(ROOT, "include"),
           "-isystem", os.path.join(ROCM, "include"), "-x", "c++", os.path.join(CSRC, "bdrs_api.hip"),
           os.path.join(ROOT, "tests", "api_driver.cpp"), "-o", exe]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    return exe


@pytest.mark.parametrize("scenario", ["results_are_there", "refused_under_capture", "weights_after_an_error",
                                      "weights_after_a_numeric_error", "weights_after_a_capture"])
def test_host_side(driver, scenario):
    res = subprocess.run([driver, scenario], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0 and res.stdout.strip().endswith("ok"), res.stdout + res.stderr
