"""Regions of the workspace that the iterative assignment uses, and the workspace's size at the largest problem (no GPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2508_12801_amd", "csrc")
SAN = os.path.join(ROOT, "tests", "sanitize")


def test_iterative_assignment_fits(tmp_path):
    clang = "/opt/rocm/llvm/bin/clang++"
    if not os.path.exists(clang):
        clang = shutil.which("clang++") or shutil.which("g++")
    if clang is None or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("no host compiler or HIP headers")
    exe = str(tmp_path / "workspace")
    subprocess.check_call([clang, "-std=c++17", "-x", "c++", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", os.path.join(ROOT, "include"),
                           "-I", CSRC, os.path.join(CSRC, "api.cpp"), os.path.join(SAN, "host_stubs.cpp"),
                           os.path.join(SAN, "workspace_driver.cpp"), "-o", exe])
    r = subprocess.run([exe], stdout=subprocess.PIPE, text=True)
    print(r.stdout)
    assert r.returncode == 0, r.stdout


def test_the_last_rerouting_rounds_fit_one_launch(tmp_path):
    exe = str(tmp_path / "iter_tail")
    subprocess.check_call(["g++", "-std=c++17", "-I", CSRC, os.path.join(SAN, "iter_tail.cpp"), "-o", exe])
    r = subprocess.run([exe], stdout=subprocess.PIPE, text=True)
    assert r.returncode == 0, r.stdout
