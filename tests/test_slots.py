"""Rounds of few (request, KV head) pairs, which split a request into more than 32 slots.

CPU: workspace sizes on both sides of the rule, and the planner's checks on
such rounds.  GPU: parity with the fp64 oracle where finalize merges 33 to 128
slots, for narrow and wide query groups, batched and per-chunk (merged into
slots already written), with a caller's workspace and the library's scratch.
"""
from __future__ import annotations

import os
import shutil
import subprocess

import pytest
import torch

from paper_2609_33184_amd import harness as H
from paper_2609_33184_amd import specstream as ss
from paper_2609_33184_amd import workloads as W
from parity import assert_parity, oracle_full

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("cand,heads,slots", [([8], (8, 1), 128), ([8, 1], (8, 1), 128), ([5], (8, 2), 128),
                                              ([5] * 3, (8, 1), 64), ([6], (32, 4), 64), ([6], (24, 3), 64),
                                              ([6, 6], (8, 2), 64), ([6] * 5, (8, 1), 32), ([6] * 3, (8, 2), 32),
                                              ([5], (32, 8), 32), ([5], (5, 5), 32)])
def test_workspace_slots(cand, heads, slots):
    up = lambda x: (x + 255) // 256 * 256
    rows = sum(cand) * heads[0] * slots
    want = up(rows * 128 * 4) + 2 * up(rows * 4) + 256
    assert ss.ss_round_workspace_bytes(ss.make_desc(cand, *heads)) == want
    assert want <= 64 << 20       # the scratch still serves such a round


def test_planner_few_pairs(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None or not os.path.exists("/opt/rocm/lib/libamdhip64.so"):
        pytest.skip("needs g++ and the ROCm runtime library to link the host code")
    exe = tmp_path / "plan_few_pairs"
    subprocess.run([cxx, "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", f"-I{ROOT}/include",
                    f"-I{ROOT}/paper_2609_33184_amd/csrc", os.path.join(ROOT, "tests", "cpp", "plan_few_pairs.cpp"),
                    os.path.join(ROOT, "paper_2609_33184_amd", "csrc", "ss_host.cpp"), "-L/opt/rocm/lib", "-lamdhip64",
                    "-Wl,-rpath,/opt/rocm/lib", "-o", str(exe)], check=True, capture_output=True, text=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0 and "all ok" in res.stdout, res.stdout[-3000:] + res.stderr[-2000:]


CASES = [  # heads, history lengths, candidates, chunk tokens, chunks per call
    ((2, 2), [17000], [5], 4096, 5),                 # 33 slots
    ((8, 4), [32768], [4], 4096, 8),                 # 64
    ((32, 4), [32790], [6], 5000, 7),                # 64, wide query group
    ((4, 2), [65536], [8], 8192, 8),                 # 128
    ((3, 1), [40000, 30001], [7, 1], 9000, 5),       # two requests
    ((8, 1), [50000, 0, 1, 20000], [8, 8, 3, 1], 25000, 1),   # per-chunk calls, wide, an empty history
    ((6, 1), [66000], [1], 33000, 1),
]


@pytest.mark.gpu
@pytest.mark.parametrize("scratch", [False, True])
@pytest.mark.parametrize("heads,lens,cands,chunk,batch", CASES)
def test_many_slots(heads, lens, cands, chunk, batch, scratch):
    w = W.custom(lens, cands, num_q_heads=heads[0], num_kv_heads=heads[1], chunk_tokens=chunk, seed_base=77)
    b = H.RoundBuffers(w)
    b.out.fill_(float("nan"))
    chunks = H.hbm_history(w)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    H.run_round(b, chunks, s.cuda_stream, batch=batch, scratch=scratch)
    s.synchronize()
    ref_o, ref_l = _oracle(w)
    assert_parity(b.out.double().cpu().numpy(), ref_o, f"{heads} {lens}", rel_l2=1e-5)
    assert_parity(b.lse.double().cpu().numpy(), ref_l, "lse", max_abs=1e-4, rel_l2=1e-5)


def test_workspace_of_a_larger_cohort():
    """Fewer requests may ask for more slots, and run on what the larger cohort's workspace holds."""
    heads = (16, 2)
    need = lambda n: ss.ss_round_workspace_bytes(ss.make_desc([8] * n, *heads))
    held = need(3)
    assert held < need(2) == 64 * 256 * 520 + 256 and held < need(1) == 128 * 128 * 520 + 256
    for n in (3, 2, 1):
        ss.ss_round_destroy(ss.ss_round_init(ss.make_desc([8] * n, *heads), 0x7f0000000000, 0x7f1000000000, held))
        base = 32 * 128 * n * 520 + 256          # 32 slots: the least that a round takes
        for enough in (base, max(base, need(n) - 257), max(base, need(n) - 20000)):
            ss.ss_round_destroy(ss.ss_round_init(ss.make_desc([8] * n, *heads), 0x7f0000000000, 0x7f1000000000, enough))
        for short in (base - 1, need(n) - 1, need(n) - 256):
            with pytest.raises(ss.SpecStreamError) as e:
                ss.ss_round_init(ss.make_desc([8] * n, *heads), 0x7f0000000000, 0x7f1000000000, short)
            assert e.value.status == ss.SS_ERR_WORKSPACE


@pytest.mark.parametrize("heads", [(1, 1), (2, 2), (3, 3), (4, 4), (15, 3), (16, 2), (64, 1), (32, 4)])
def test_every_larger_cohorts_workspace_serves(heads):
    """Any cohort runs on the workspace of any cohort of the same heads with as many candidates or more."""
    need = lambda cand: ss.ss_round_workspace_bytes(ss.make_desc(cand, *heads))
    cohorts = [[n] * b for b in (1, 2, 3, 4, 5, 8) for n in (1, 3, 5, 8) if n * heads[0] // heads[1] <= 64]
    for small in cohorts:
        for large in cohorts:
            if len(large) >= len(small) and sum(large) >= sum(small):
                ss.ss_round_destroy(ss.ss_round_init(ss.make_desc(small, *heads), 0x7f0000000000, 0x7f1000000000, need(large)))


@pytest.mark.gpu
@pytest.mark.parametrize("slots", [32, 64])
def test_fewer_slots_than_asked_for(slots):
    """1 x 40000 tokens, 2 KV heads: 78 shares with 128 slots, 64 or 32 on smaller workspaces."""
    w = W.custom([40000], [7], num_q_heads=6, num_kv_heads=2, chunk_tokens=8192, seed_base=78)
    b = H.RoundBuffers(w)
    up = lambda x: (x + 255) // 256 * 256
    b.ws_bytes = up(42 * slots * 512) + 2 * up(42 * slots * 4) + 256
    b.ws = torch.full((b.ws_bytes + 4096,), 0xFF, dtype=torch.uint8, device="cuda")   # NaN states
    b.out.fill_(float("nan"))
    chunks = H.hbm_history(w)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    H.run_round(b, chunks, s.cuda_stream, batch=5)
    s.synchronize()
    assert bool((b.ws[b.ws_bytes:] == 0xFF).all())
    ref_o, ref_l = _oracle(w)
    assert_parity(b.out.double().cpu().numpy(), ref_o, f"{slots} slots", rel_l2=1e-5)
    assert_parity(b.lse.double().cpu().numpy(), ref_l, "lse", max_abs=1e-4, rel_l2=1e-5)


@pytest.mark.gpu
def test_one_zeroed_workspace_for_every_cohort():
    """Cohorts of other sizes and slot counts take turns on one zero-filled workspace; their claim counter stays
    zero, so balanced rounds equal, bitwise, the same rounds on workspaces of their own."""
    cohorts = [W.custom(lens, cands, num_q_heads=8, num_kv_heads=2, chunk_tokens=65536, seed_base=79)
               for lens, cands in [([200000] * 3, [8] * 3), ([300000, 262144], [5, 2]), ([262144] * 4, [8, 1, 2, 3])]]
    s = torch.cuda.Stream()
    rounds = []
    for w in cohorts:
        chunks = H.hbm_history(w)
        b = H.RoundBuffers(w, balance_permille=100)
        torch.cuda.synchronize()
        H.run_round(b, chunks, s.cuda_stream, batch=8)
        s.synchronize()
        rounds.append((w, chunks, b.out.clone(), b.lse.clone(), b.ws_bytes))
    held = torch.zeros(max(r[4] for r in rounds) + 1000, dtype=torch.uint8, device="cuda")
    for _ in range(2):
        for w, chunks, out, lse, _ in rounds:
            b = H.RoundBuffers(w, balance_permille=100, counters_zeroed=1)
            b.ws, b.ws_bytes = held, held.numel()
            torch.cuda.synchronize()
            H.run_round(b, chunks, s.cuda_stream, batch=8)
            s.synchronize()
            assert torch.equal(b.out, out) and torch.equal(b.lse, lse), f"{w.B} requests"
            counters = held[held.numel() // 256 * 256 - 256:][:256]
            assert not bool(counters.any())


_CACHE = {}


def _oracle(w):
    key = (w.num_q_heads, w.num_kv_heads, tuple(w.hist_len), tuple(w.num_cand))
    if key not in _CACHE:
        _CACHE[key] = oracle_full(w)
    return _CACHE[key]
