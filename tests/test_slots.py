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


_CACHE = {}


def _oracle(w):
    key = (w.num_q_heads, w.num_kv_heads, tuple(w.hist_len), tuple(w.num_cand))
    if key not in _CACHE:
        _CACHE[key] = oracle_full(w)
    return _CACHE[key]
