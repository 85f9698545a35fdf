"""The device pool's host code, without a GPU: blocks of a thread that ends while the
device is being waited for are not handed out before the next wait."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_blocks_handed_over_during_a_wait_stay_back(tmp_path):
    gxx = shutil.which("g++")
    inc = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")
    if not gxx or not os.path.isdir(inc):
        pytest.skip("no host compiler or HIP headers")
    exe = str(tmp_path / "pool_idle_driver")
    subprocess.run([gxx, "-std=c++17", "-g", "-D__HIP_PLATFORM_AMD__", "-I", inc,
                    "-o", exe, os.path.join(ROOT, "tests", "pool_idle_driver.cpp"), "-pthread"],
                   check=True, capture_output=True, text=True, timeout=300)
    assert subprocess.run([exe], timeout=60).returncode == 0
