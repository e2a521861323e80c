"""plan.cpp over a stand-in HIP runtime (tests/host/runtime.cpp): what a call hands to
its kernel and what a plan takes of the device's memory, without a device.

Compiled with g++ and the undefined-behaviour sanitizer; each check is one run of the
program.
"""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
ROCM = "/opt/rocm"


@pytest.fixture(scope="module")
def checks(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.exists(os.path.join(ROCM, "include", "hip", "hip_runtime_api.h")):
        pytest.skip("needs g++ and the HIP headers")
    exe = str(tmp_path_factory.mktemp("host") / "runtime_checks")
    src = [os.path.join(ROOT, "paper_2204_00602_amd", "csrc", "plan.cpp"),
           os.path.join(HERE, "host", "runtime.cpp"), os.path.join(HERE, "host", "runtime_checks.cpp")]
    subprocess.run([gxx, "-std=c++17", "-O1", "-g", "-fsanitize=undefined", "-fno-sanitize-recover=undefined",
                    "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"), "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2204_00602_amd", "csrc"), "-I", os.path.join(HERE, "host")] + src +
                   ["-o", exe, "-ldl", "-lpthread"], check=True, timeout=600)
    return exe


@pytest.mark.parametrize("name", [
    "select-threads",  # a call whose helper threads cannot be started, after calls that had some
    "select-parts",    # every multiset of occupations beside a small one
    "table-memory",    # plans, batches and sources in the memory they take without tables
    "noalloc-area",    # plans that slos_amplitudes_noalloc takes without tables
    "allocation-failures",  # each host allocation of a call failing in turn
])
def test_host_runtime(checks, name):
    res = subprocess.run([checks, name], capture_output=True, text=True, timeout=600)
    assert res.returncode == 0, res.stdout[-4000:] + res.stderr[-2000:]
