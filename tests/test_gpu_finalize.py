"""The finalize kernel's builds and dispatch against the fp64 oracle.

A launch picks a build by the largest slot count (8, 16 or 32), splits a
row's slots and candidates over a workgroup's waves when few workgroups run,
splits the candidates over launches beyond its table, and addresses each slot
by itself once the slots pass 2^32 bytes.  Head counts that do not fill a
workgroup's last pair or block of heads, every kind of query-group division,
requests without history and slot counts on both sides of each build are
drawn in; the bar is that of the other parity tests.
"""
from __future__ import annotations

import pytest
import torch

from paper_2609_33184_amd import harness as H
from paper_2609_33184_amd import specstream as ss
from paper_2609_33184_amd import workloads as W
from parity import assert_parity, oracle_full

# name, heads, history lengths, candidates, tokens per share
CASES = [
    ("one head, one candidate, no history", (1, 1), [0], [1], 32),
    ("odd heads, 1 slot", (3, 3), [7, 32], [8, 1], 0),
    ("G = 3, 8 slots", (6, 2), [256, 40, 0], [5, 8, 2], 32),
    ("G = 5, 9 slots", (15, 3), [288, 33], [8, 3], 32),
    ("G = 7, 16 and 17 slots", (7, 1), [512, 544, 1], [8, 7, 8], 32),
    ("G = 4, 31 and 32 slots", (32, 8), [1024, 992], [4, 8], 32),
    ("rows not split (over 1024 pairs)", (32, 8), [100 + i for i in range(20)], [8 - i % 8 for i in range(20)], 32),
    ("rows not split, 17 slots", (48, 8), [544] + [32] * 9, [8] * 10, 32),
    ("heads past a block of 8, not split", (10, 2), [64] * 40, [8] * 40, 32),
    ("candidates over one table", (1, 1), [1 + i % 40 for i in range(520)], [8] * 520, 0),
    ("slots past 2^32 bytes", (32, 8), [i % 3 for i in range(1025)], [8] * 1025, 0),
]


@pytest.mark.gpu
@pytest.mark.parametrize("name,heads,lens,cands,split", CASES, ids=[c[0] for c in CASES])
def test_finalize(name, heads, lens, cands, split):
    w = W.custom(lens, cands, num_q_heads=heads[0], num_kv_heads=heads[1], chunk_tokens=2048, seed_base=31)
    print(name, flush=True)
    b = H.RoundBuffers(w, split_tokens=split)
    b.out.fill_(float("nan"))
    b.lse.fill_(float("nan"))
    chunks = H.hbm_history(w)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    H.run_round(b, chunks, s.cuda_stream)
    s.synchronize()
    ref_o, ref_l = oracle_full(w)
    assert_parity(b.out.double().cpu().numpy(), ref_o, name)
    assert float(abs(b.lse.double().cpu().numpy() - ref_l).max()) <= 1e-3
