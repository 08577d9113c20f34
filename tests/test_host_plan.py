"""What a plan holds on the host (tests/sanitize/plan_driver.cpp), with the library's host half built by the host
C++ compiler and the device launchers replaced by stand-ins."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2110_11866_amd", "csrc")
HERE = os.path.join(ROOT, "tests", "sanitize")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def test_plan_state(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None or not os.path.isdir(os.path.join(ROCM, "include", "hip")):
        pytest.skip("needs g++ and the HIP headers")
    exe = str(tmp_path / "plan_driver")
    subprocess.run([cxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"),
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(CSRC, "plan.cpp"), os.path.join(HERE, "host_stubs.cpp"),
                    os.path.join(HERE, "plan_driver.cpp"), "-L", os.path.join(ROCM, "lib"),
                    "-Wl,-rpath," + os.path.join(ROCM, "lib"), "-lamdhip64", "-o", exe],
                   check=True, capture_output=True, text=True)
    env = dict(os.environ, HIP_VISIBLE_DEVICES="")
    r = subprocess.run([exe], capture_output=True, text=True, env=env, timeout=300)
    assert r.returncode == 0 and "all checks passed" in r.stdout, r.stdout + r.stderr
