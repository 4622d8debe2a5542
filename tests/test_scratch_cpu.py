"""What a thread keeps between history calls (tests/cpp/scratch_check.cpp), checked on the CPU.

The planner's tables stay allocated from call to call, so that ordinary calls
allocate nothing, and are given back after a call that needed much more.
"""
from __future__ import annotations

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_planner_memory_is_bounded(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None or not os.path.exists("/opt/rocm/lib/libamdhip64.so"):
        pytest.skip("needs g++ and the ROCm runtime library to link the host code")
    exe = tmp_path / "scratch_check"
    subprocess.run([cxx, "-O1", "-std=c++17", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    f"-I{ROOT}/include", f"-I{ROOT}/paper_2609_33184_amd/csrc",
                    os.path.join(ROOT, "tests", "cpp", "scratch_check.cpp"),
                    os.path.join(ROOT, "paper_2609_33184_amd", "csrc", "ss_host.cpp"), "-L/opt/rocm/lib", "-lamdhip64",
                    "-Wl,-rpath,/opt/rocm/lib", "-o", str(exe)], check=True, capture_output=True, text=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0 and "all ok" in res.stdout, res.stdout[-3000:] + res.stderr[-2000:]
