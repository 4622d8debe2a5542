"""Uploads copy exactly the bytes asked for, by kernel or by copy engine.

Sizes lie on both sides of a 16-byte word, of the kernel's block and of its
size limit; sources and destinations start at aligned and unaligned offsets
of larger buffers (the kernel takes 16-byte-aligned ones).  The bytes around
the destination stay as they were, and an upload captured in a HIP graph
copies what the source holds at each replay.
"""
from __future__ import annotations

import pytest
import torch

from paper_2609_33184_amd import specstream as ss

KERNEL_BLOCK = 256 * 4 * 16
LIMIT = 64 << 20


def _bytes(n, seed):
    g = torch.Generator().manual_seed(seed)
    return torch.randint(0, 256, (n,), dtype=torch.uint8, generator=g).pin_memory()


@pytest.mark.gpu
@pytest.mark.parametrize("src_off,dst_off", [(0, 0), (16, 48), (1, 0), (0, 8), (7, 7)])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 4095, KERNEL_BLOCK - 1, KERNEL_BLOCK, KERNEL_BLOCK + 16,
                               17 * KERNEL_BLOCK + 33, LIMIT, LIMIT + 1])
def test_upload_bytes(n, src_off, dst_off):
    ss.load()
    if n >= LIMIT and src_off not in (0, 1):
        pytest.skip("large sizes: one aligned and one unaligned start")
    src = _bytes(n + src_off, n % 1000 + src_off)
    dst = torch.full((n + dst_off + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    ss.ss_upload_chunk(dst.data_ptr() + dst_off, src.data_ptr() + src_off, n, s.cuda_stream)
    s.synchronize()
    got = dst.cpu()
    assert torch.equal(got[dst_off:dst_off + n], src[src_off:])
    assert bool((got[:dst_off] == 0xA5).all()) and bool((got[dst_off + n:] == 0xA5).all())


@pytest.mark.gpu
def test_upload_in_a_graph():
    ss.load()
    n = 5 * KERNEL_BLOCK + 40
    src, dst = _bytes(n, 3), torch.zeros(n, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        ss.ss_upload_chunk(dst.data_ptr(), src.data_ptr(), n, torch.cuda.current_stream().cuda_stream)
    for k in range(3):
        src.copy_(_bytes(n, 10 + k))
        dst.fill_(k)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(dst.cpu(), src)
