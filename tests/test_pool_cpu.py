"""The device pool's host code, without a GPU, under AddressSanitizer: buffers that a
thread keeps for its life are released as it ends, in whatever order its other
per-thread data goes, and their blocks serve the next thread."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_buffers_released_as_a_thread_ends(tmp_path):
    gxx = shutil.which("g++")
    inc = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")
    if not gxx or not os.path.isdir(inc):
        pytest.skip("no host compiler or HIP headers")
    exe = str(tmp_path / "pool_exit_driver")
    subprocess.run([gxx, "-std=c++17", "-g", "-fsanitize=address", "-D__HIP_PLATFORM_AMD__", "-I", inc,
                    "-o", exe, os.path.join(ROOT, "tests", "pool_exit_driver.cpp"), "-pthread"],
                   check=True, capture_output=True, text=True, timeout=300)
    env = {k: v for k, v in os.environ.items() if k != "LD_PRELOAD"}
    env["ASAN_OPTIONS"] = "detect_leaks=0"
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120, env=env)
    assert r.returncode == 0, r.stderr[-2000:]
