"""Short shares that span requests: launches with a workgroup per unit and with
one per share, on both sides of the rule between them, against the fp64 oracle
and bitwise against a repeat of the round.

A share's units differ in request, row count and so in kernel body; some
requests have no history, some workgroups no unit of their own.
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2609_33184_amd import harness as H
from paper_2609_33184_amd import specstream as ss
from paper_2609_33184_amd import workloads as W
from parity import assert_parity, oracle_full

# heads, requests, longest history, tokens per share (0 = automatic), chunk tokens, chunks per call
CASES = [
    ((8, 8), 24, 300, 0, 1024, 1),
    ((32, 8), 24, 900, 0, 200, 8),          # chains over chunk boundaries
    ((32, 8), 20, 1500, 256, 1024, 2),      # 8 tiles a share: a workgroup per unit
    ((32, 8), 20, 1500, 288, 1024, 2),      # 9 tiles: a workgroup per share
    ((16, 8), 70, 300, 128, 1024, 1),       # over 768 units
    ((64, 8), 12, 700, 0, 1024, 1),         # 1 to 4 row blocks mixed
    ((12, 2), 90, 120, 32, 64, 2),          # shares of one tile, workgroups without units
]


@pytest.mark.gpu
@pytest.mark.parametrize("heads,requests,longest,split,chunk,batch", CASES)
def test_short_shares(heads, requests, longest, split, chunk, batch):
    rng = np.random.default_rng(requests + longest + split)
    lens = [0 if rng.random() < 0.1 else int(rng.integers(1, longest + 1)) for _ in range(requests)]
    cands = [int(rng.integers(1, 9)) for _ in range(requests)]
    w = W.custom(lens, cands, num_q_heads=heads[0], num_kv_heads=heads[1], chunk_tokens=chunk, seed_base=91)
    b = H.RoundBuffers(w, split_tokens=split)
    chunks = H.hbm_history(w)
    s = torch.cuda.Stream()
    outs = []
    for _ in range(2):
        b.out.fill_(float("nan"))
        torch.cuda.synchronize()
        H.run_round(b, chunks, s.cuda_stream, batch=batch)
        s.synchronize()
        outs.append((b.out.clone(), b.lse.clone()))
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
    ref_o, ref_l = oracle_full(w)
    assert_parity(outs[0][0].double().cpu().numpy(), ref_o, f"{heads} {requests} requests split {split}", rel_l2=1e-5)
    assert_parity(outs[0][1].double().cpu().numpy(), ref_l, "lse", max_abs=1e-4, rel_l2=1e-5)
