"""The runtime (workspace, tables, streams and events; csrc/runtime.cpp) on the
CPU: tests/runtime_host_test.cpp drives its C ABI against a model of HIP's
streams, events and memory, which reports unordered uses of one workspace
block, waits of the host and tables that a launch misses."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
CASES = ["outgrown_block", "many_streams", "captured", "failed_launch", "device_full", "beside_serving", "mixed_batch", "tables", "tight_budget",
         "noalloc_tables"]


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.exists(os.path.join(ROCM, "include", "hip", "hip_runtime.h")):
        pytest.skip("no host C++ compiler or HIP headers")
    out = str(tmp_path_factory.mktemp("runtime") / "runtime_host_test")
    subprocess.run(["g++", "-std=c++20", "-O0", "-w", "-I", os.path.join(ROCM, "include"),
                    os.path.join(HERE, "runtime_host_test.cpp"), "-o", out], check=True)
    return out


@pytest.mark.parametrize("case", CASES)
def test_runtime(exe, case):
    r = subprocess.run([exe, case], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
