"""The row-split body (33 to 64 rows per KV head) at its edges, against the fp64 oracle.

A step attends two 32-token tiles, so histories end in the first tile of a
step, in its second, inside a tile and one token past it; rows fill one, part
of or both 32-row blocks; chains cross chunk boundaries inside and between
tiles; per-chunk calls merge into slots already written.

Bound: the weights enter the product with V as two bf16 parts (2^-17 of each
weight), everything else is float32 over at most a few hundred terms, so the
relative L2 error stays below 1e-5 (2e-6 measured on long histories).
"""
from __future__ import annotations

import pytest
import torch

from paper_2609_33184_amd import harness as H
from paper_2609_33184_amd import specstream as ss
from paper_2609_33184_amd import workloads as W
from parity import assert_parity, oracle_full

LENS = [1, 31, 32, 33, 63, 64, 65, 96, 97, 128, 129, 300]
ROWS = [(8, 8), (8, 5), (6, 6), (6, 8), (11, 3), (13, 4)]   # query heads per KV head, candidates: 64, 40, 36, 48, 33, 52 rows


@pytest.mark.gpu
@pytest.mark.parametrize("layout", [ss.SS_KV_TOKEN_MAJOR, ss.SS_KV_HEAD_MAJOR, ss.SS_KV_HEAD_MAJOR_KV])
@pytest.mark.parametrize("chunk,batch,split", [(512, 1, 0), (40, 8, 0), (40, 1, 0), (512, 1, 64), (96, 4, 96)])
@pytest.mark.parametrize("group,cand", ROWS)
def test_row_split_edges(group, cand, chunk, batch, split, layout):
    w = W.custom(LENS, [cand] * len(LENS), num_q_heads=2 * group, num_kv_heads=2, chunk_tokens=chunk, seed_base=57)
    b = H.RoundBuffers(w, split_tokens=split, kv_layout=layout)
    b.out.fill_(float("nan"))
    chunks = H.hbm_history(w, kv_layout=layout)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    H.run_round(b, chunks, s.cuda_stream, batch=batch)
    s.synchronize()
    ref_o, ref_l = _oracle(w)
    what = f"G={group} n={cand} chunk={chunk} batch={batch} split={split} layout={layout}"
    assert_parity(b.out.double().cpu().numpy(), ref_o, what, rel_l2=1e-5)
    assert_parity(b.lse.double().cpu().numpy(), ref_l, what + " lse", max_abs=1e-4, rel_l2=1e-5)


_CACHE = {}


def _oracle(w):
    key = (w.num_q_heads, tuple(w.num_cand))    # the history does not depend on the chunking
    if key not in _CACHE:
        _CACHE[key] = oracle_full(w)
    return _CACHE[key]


@pytest.mark.gpu
@pytest.mark.parametrize("group,cand", [(8, 8), (6, 8), (5, 7)])
@pytest.mark.parametrize("masked", [(32, 64), (0, 32), (32, 96), (0, 100)])
def test_keys_of_minus_infinity(group, cand, masked):
    """A whole tile of scores at -inf weighs nothing, whichever wave attends it first.

    Queries are positive, so a key of -inf scores -inf for every row; the
    tokens [lo, hi) of each request have such keys.
    """
    lens, lo, hi = [100, 64, 131], *masked
    w = W.custom(lens, [cand] * len(lens), num_q_heads=group, num_kv_heads=1, chunk_tokens=256, seed_base=58)
    b = H.RoundBuffers(w)
    b.q.abs_().clamp_(min=0.01)
    b.out.fill_(float("nan"))
    (k, v), = H.hbm_history(w)
    starts = [sum(lens[:i]) for i in range(len(lens))]
    for s0, n in zip(starts, lens):
        k[s0 + lo:s0 + min(hi, n)] = float("-inf")
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    H.run_round(b, [(k, v)], s.cuda_stream)
    s.synchronize()
    for i, n in enumerate(lens):
        r = slice(i * cand, (i + 1) * cand)
        q = b.q[r].double().reshape(cand * group, 128)
        keys = torch.cat([k[starts[i]:starts[i] + n, 0], b.kc[r, 0]]).double()
        vals = torch.cat([v[starts[i]:starts[i] + n, 0], b.vc[r, 0]]).double()
        seen = torch.cat([torch.ones(cand, n, device="cuda"), torch.ones(cand, cand, device="cuda").tril()], 1).bool()
        # not a matrix product: 0 x inf has no part in the scores
        x = (q[:, None, :] * keys[None]).sum(-1) * w.softmax_scale
        x = x.masked_fill(~seen.repeat_interleave(group, 0), float("-inf"))
        ref = torch.softmax(x, 1) @ vals
        what = f"G={group} n={cand} request {i} masked {masked}"
        assert_parity(b.out[r].double().reshape(cand * group, 128).cpu().numpy(), ref.cpu().numpy(), what, rel_l2=1e-5)
        assert_parity(b.lse[r].double().reshape(-1).cpu().numpy(), torch.logsumexp(x, 1).cpu().numpy(), what + " lse",
                      max_abs=1e-4, rel_l2=1e-5)
