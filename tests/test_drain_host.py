"""The drain's bounds and errors (CPU only): tests/drain_driver.cpp runs
gsys_wait, gsys_stats_get, gsys_unregister_buffer and gsys_shutdown of a
device context over a device that does not hand the ticket counter over, hands
it over late, or fails."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1705_06965_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    gxx = shutil.which("g++")
    if not gxx or not os.path.exists(os.path.join(ROCM, "include", "hip", "hip_runtime.h")):
        pytest.skip("g++ or the HIP headers are missing")
    exe = str(tmp_path_factory.mktemp("drain") / "drain_driver")
    cmd = [gxx, "-std=c++17", "-O1", "-g", "-D__HIP_PLATFORM_AMD__", "-w",
           "-I" + os.path.join(ROCM, "include"), "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
           os.path.join(ROOT, "tests", "drain_driver.cpp"), os.path.join(CSRC, "capi.cpp"),
           os.path.join(CSRC, "host_pool.cpp"), "-o", exe, "-L" + os.path.join(ROCM, "lib"),
           "-lamdhip64", "-lhsa-runtime64", "-pthread", "-Wl,-rpath," + os.path.join(ROCM, "lib")]
    b = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert b.returncode == 0, b.stderr[-3000:]
    return exe


@pytest.mark.parametrize("what", ["never", "late", "errors", "release_read", "release_never",
                                  "release_fails"])
def test_drain(driver, what):
    r = subprocess.run([driver, what], capture_output=True, text=True, timeout=40)
    assert r.returncode == 0, r.stdout + r.stderr
