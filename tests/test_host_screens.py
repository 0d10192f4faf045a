"""The host's check of Jones fields, built and run on the CPU (tests/screen_check_driver.cpp)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(ROOT, "paper_2206_15117_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.exists(os.path.join(ROCM, "include", "hip", "hip_runtime.h")):
        pytest.skip("g++ or the HIP headers are not installed")
    exe = str(tmp_path_factory.mktemp("screens") / "driver")
    res = subprocess.run(["g++", "-std=c++17", "-O2", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROOT, "include"),
                          "-I", CSRC, "-I", os.path.join(ROCM, "include"), os.path.join(CSRC, "mueller.cpp"),
                          os.path.join(HERE, "screen_check_driver.cpp"), "-o", exe, "-L", os.path.join(ROCM, "lib"),
                          "-lamdhip64", "-Wl,-rpath," + os.path.join(ROCM, "lib")], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    return exe


def test_accepted_fields_have_finite_screens(driver):
    res = subprocess.run([driver], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stdout + res.stderr


def test_the_threads_allocate_nothing(driver):
    """Memory that runs out inside a worker thread would end the process: allocations there throw in this run."""
    res = subprocess.run([driver, "threads"], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stdout + res.stderr
