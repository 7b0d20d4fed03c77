"""The host side of the ABI where a launch fails: grawa_api.cpp and grawa_maps.cpp built for the CPU, the HIP runtime and the
kernels replaced by stubs (tests/api_host_driver.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM_INCLUDE = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")
pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(ROCM_INCLUDE), reason="no host compiler or HIP headers")


def test_failed_launches(tmp_path):
    csrc = os.path.join(ROOT, "paper_2403_04206_amd", "csrc")
    out = str(tmp_path / "driver")
    res = subprocess.run(["g++", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I", ROCM_INCLUDE, "-I", os.path.join(ROOT, "include"),
                          "-I", csrc, os.path.join(ROOT, "tests", "api_host_driver.cpp"), os.path.join(csrc, "grawa_api.cpp"),
                          os.path.join(csrc, "grawa_maps.cpp"), "-o", out], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    res = subprocess.run([out], capture_output=True, text=True, timeout=60)
    assert res.returncode == 0 and res.stdout.strip() == "ok", res.stdout
