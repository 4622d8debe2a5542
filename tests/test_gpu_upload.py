"""Uploads copy exactly the bytes asked for, by copy engine or by kernel.

ss_upload_chunk (copy engine) takes sizes from one byte past 64 MiB, from
aligned and unaligned offsets of larger buffers.  The pipeline's uploads take
sizes on both sides of the upload kernel's block, of its grid and of its size
limit, from offsets that it takes and that it leaves to the engine, and
sources of every kind of pinned memory, rewritten between uploads.  The bytes
around the destination stay as they were, and an upload captured in a HIP
graph copies what the source holds at each replay.
"""
from __future__ import annotations

import ctypes

import pytest
import torch

from paper_2609_33184_amd import specstream as ss

BLOCK = 256 * 4 * 16
LARGE = 64 << 20


def _bytes(n, seed):
    g = torch.Generator().manual_seed(seed)
    return torch.randint(0, 256, (n,), dtype=torch.uint8, generator=g).pin_memory()


@pytest.mark.gpu
@pytest.mark.parametrize("src_off,dst_off", [(0, 0), (16, 48), (1, 0), (0, 8), (7, 7)])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 4095, BLOCK - 1, BLOCK, BLOCK + 16,
                               17 * BLOCK + 33, LARGE, LARGE + 1])
def test_upload_bytes(n, src_off, dst_off):
    ss.load()
    if n >= LARGE and src_off not in (0, 1):
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
    n = 5 * BLOCK + 40
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


TOKEN = 512             # bytes of a token's K and V, one KV head


class _Pipe:
    """A pipeline over two guarded staging slots and rounds of one request, one KV head and one candidate."""

    def __init__(self, nbytes, copy_stream, stream):
        self.stream, self.nbytes = stream, nbytes
        self.slots = [torch.full((nbytes + 256,), 0xA5, dtype=torch.uint8, device="cuda") for _ in range(2)]
        self.p = ss.ss_pipeline_create(self.slots[0].data_ptr(), self.slots[1].data_ptr(), nbytes, copy_stream.cuda_stream)
        self.q = torch.randn(1, 1, 128, device="cuda").to(torch.bfloat16)
        self.desc = ss.make_desc([1], 1, 1, max_chunk_tokens=nbytes // TOKEN)
        self.ws = torch.zeros(ss.ss_round_workspace_bytes(self.desc), dtype=torch.uint8, device="cuda")
        self.out = torch.empty(1, 1, 128, device="cuda")

    def round(self, sources):
        s = self.stream.cuda_stream
        r = ss.ss_round_init(self.desc, self.q.data_ptr(), self.ws.data_ptr(), self.ws.numel(), s)
        for src in sources:
            ss.ss_pipeline_attend_chunk(self.p, r, src, [self.nbytes // TOKEN], s)
        ss.ss_attend_local_candidates(r, self.q.data_ptr(), self.q.data_ptr(), s)
        ss.ss_round_finalize(r, self.out.data_ptr(), None, s)
        ss.ss_round_destroy(r)

    def close(self):
        torch.cuda.synchronize()
        ss.ss_pipeline_destroy(self.p)


@pytest.mark.gpu
@pytest.mark.parametrize("off", [0, 16, 4])
@pytest.mark.parametrize("tokens", [1, 31, 32, 33, 65, 16 * 16 + 1, 16 * 32, 17 * 32 + 1, (2 << 20) // TOKEN - 1,
                                    (2 << 20) // TOKEN + 257, (4 << 20) // TOKEN + 15, (16 << 20) // TOKEN,
                                    (16 << 20) // TOKEN + 1])
def test_pipeline_upload_bytes(tokens, off):
    ss.load()
    n = tokens * TOKEN
    src = [_bytes(n + off, tokens + k) for k in range(3)]
    torch.cuda.synchronize()
    p = _Pipe(n, torch.cuda.Stream(), torch.cuda.Stream())
    p.round([x.data_ptr() + off for x in src])
    torch.cuda.synchronize()
    for slot, x in ((0, src[2]), (1, src[1])):
        got = p.slots[slot].cpu()
        assert torch.equal(got[:n], x[off:]) and bool((got[n:] == 0xA5).all())
    p.close()


@pytest.mark.gpu
@pytest.mark.parametrize("flags", [0, 1, 2, 4, 0x40000000, 0x80000000])
def test_pipeline_upload_of_rewritten_memory(flags):
    """Default, portable, mapped, write-combined, coherent and non-coherent hipHostMalloc memory."""
    ss.load()
    hip = ctypes.CDLL("libamdhip64.so")
    n = 100 * TOKEN
    ptr = ctypes.c_void_p()
    assert hip.hipHostMalloc(ctypes.byref(ptr), ctypes.c_size_t(n), ctypes.c_uint(flags)) == 0
    torch.cuda.synchronize()
    p = _Pipe(n, torch.cuda.Stream(), torch.cuda.Stream())
    for k in range(6):
        x = _bytes(n, 40 + k)
        ctypes.memmove(ptr.value, x.data_ptr(), n)
        p.round([ptr.value])
        p.stream.synchronize()
        assert torch.equal(p.slots[k % 2].cpu()[:n], x), f"upload {k}"
    p.close()
    assert hip.hipHostFree(ptr) == 0


@pytest.mark.gpu
def test_pipeline_upload_in_a_graph():
    ss.load()
    n = 165 * TOKEN
    src = _bytes(n, 3)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    p = _Pipe(n, s, s)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        p.round([src.data_ptr()])
    for k in range(3):
        src.copy_(_bytes(n, 20 + k))
        p.slots[0].fill_(k)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(p.slots[0].cpu()[:n], src)
    p.close()
