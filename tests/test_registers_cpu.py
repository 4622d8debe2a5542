"""Registers of the built kernels: what has to share a CU must fit, and nothing spills to memory.

A SIMD has 512 VGPRs, given out in eights.  Two workgroups of four waves put
two waves on each; a wave of the upload kernel must find room beside two of
the wide history kernel's, or uploads wait for whole launches to end.
"""
from __future__ import annotations

import os
import re
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2609_33184_amd", "libspecstream.so")
READELF = "/opt/rocm/llvm/bin/llvm-readelf"
OBJCOPY = "/opt/rocm/llvm/bin/llvm-objcopy"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """name -> metadata of every kernel in this repository's library"""
    if not (os.path.exists(LIB) and os.path.exists(READELF) and os.path.exists(OBJCOPY)):
        pytest.skip("needs the built library and the ROCm binary tools")
    d = tmp_path_factory.mktemp("fatbin")
    section = d / "fatbin"
    subprocess.run([OBJCOPY, f"--dump-section=.hip_fatbin={section}", LIB, str(d / "out.so")], check=True)
    data = section.read_bytes()
    found = {}
    for m in re.finditer(MAGIC, data):
        at = m.start()
        n, = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, p)
            target = data[p + 24:p + 24 + idlen].decode()
            p += 24 + idlen
            if "gfx950" not in target:
                continue
            elf = d / f"code{at}"
            elf.write_bytes(data[at + off:at + off + size])
            notes = subprocess.run([READELF, "--notes", str(elf)], check=True, capture_output=True, text=True).stdout
            for block in re.split(r"^  - (?=\.\w)", notes, flags=re.M)[1:]:
                name = re.search(r"\.name:\s+(_Z\S+)", block)
                if name:
                    found[name[1]] = {k: int(v) for k, v in re.findall(r"\.(vgpr_count|vgpr_spill_count|private_segment_fixed_size):\s+(\d+)", block)}
    assert found, "no gfx950 kernel in the library"
    return found


def _some(kernels, what):
    got = {k: v for k, v in kernels.items() if what in k}
    assert got, what
    return got


def _given(v):
    return (v["vgpr_count"] + 7) // 8 * 8


def test_upload_fits_beside_two_wide_history_workgroups(kernels):
    upload = max(_given(v) for v in _some(kernels, "copy_kernel").values())
    for name, v in _some(kernels, "chunk_attn_wide").items():
        assert 2 * _given(v) + upload <= 512, (name, v, upload)


def test_two_history_workgroups_fit_a_cu(kernels):
    for name, v in _some(kernels, "chunk_attn").items():
        assert 2 * _given(v) <= 512, (name, v)


def test_no_kernel_spills_to_memory(kernels):
    for name, v in kernels.items():
        assert v["vgpr_spill_count"] == 0 and v["private_segment_fixed_size"] == 0, (name, v)
