"""Which way an upload goes, kernel or copy engine, checked on the CPU.

tests/cpp/upload_check.cpp links the library's host code with stub launchers
and a stub HIP runtime that knows a table of allocations.  The kernel is for
ranges that lie whole inside one pinned and one device allocation of the copy
stream's GPU; every other range goes to the copy call, which checks it.  A
failed launch is reported and, behind an enqueued wait, fails the pipeline.
"""
from __future__ import annotations

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_33184_amd", "csrc")


def test_upload_route(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None or not os.path.exists("/opt/rocm/include/hip/hip_runtime_api.h"):
        pytest.skip("needs g++ and the HIP headers")
    exe = tmp_path / "upload_check"
    subprocess.run([cxx, "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", f"-I{ROOT}/include",
                    f"-I{CSRC}", os.path.join(ROOT, "tests", "cpp", "upload_check.cpp"),
                    os.path.join(CSRC, "ss_host.cpp"), os.path.join(CSRC, "ss_upload.cpp"), "-o", str(exe)],
                   check=True, capture_output=True, text=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0 and "all ok" in res.stdout, res.stdout[-3000:] + res.stderr[-2000:]
