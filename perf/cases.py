"""Timed cases of the verification round: what a serving loop asks of the library.

A case is one layer's round of one Cohort: init, the history (in one batched
call, one call per chunk, or streamed from pinned host memory through the
two-slot pipeline), the candidates, finalize.  ``listed`` names the ones that
stand for real use, ``draw`` gives more of the same ranges, ``prepare`` makes
what a serving loop holds before the round, ``run`` is the round, and
``exact`` is the same attention in float64 with plain torch.
"""
from __future__ import annotations

import math
import random

import torch

from paper_2609_33184_amd import specstream as ss

HEAD_DIM = 128
TOKEN_BYTES = 2 * 2 * HEAD_DIM          # K and V rows of one token and KV head, bf16
LAYOUTS = {"token": ss.SS_KV_TOKEN_MAJOR, "head": ss.SS_KV_HEAD_MAJOR, "head_kv": ss.SS_KV_HEAD_MAJOR_KV}
MAX_CALL_CHUNKS = 32                    # chunks one batched call takes
MOST_HISTORY_BYTES = 32 * 131072 * 8 * TOKEN_BYTES
MOST_STREAMED_BYTES = 128 << 20
# query and KV heads: the 7-8B layer, the 48- and 64-head targets, their half on each of two GPUs,
# the small test model, and one query head per KV head
HEADS = ((32, 8), (48, 8), (64, 8), (32, 4), (24, 4), (8, 2), (8, 8))


def _case(name, requests, tokens, cand, heads, chunk, layout, calls, **more):
    c = {"name": name, "requests": requests, "tokens_min": tokens[0], "tokens_max": tokens[1], "cand_min": cand[0],
         "cand_max": cand[1], "q_heads": heads[0], "kv_heads": heads[1], "chunk_tokens": chunk, "layout": layout,
         "calls": calls, "outlier_keys": False, "shape_seed": 4}
    c.update(more)
    return c


def listed():
    return [
        # the smallest call: one short request of a small model, where launches and latency count
        _case("one_request_4k", 1, (4096, 4096), (5, 5), (8, 2), 1024, "token", "batched"),
        # one interactive user of a 7-8B model at the shorter of the usual long contexts
        _case("one_request_16k", 1, (16384, 16384), (5, 5), (32, 8), 2048, "head_kv", "batched"),
        # one interactive user of the 64-head target split over two GPUs: 32 query and 4 KV heads on each
        _case("one_request_32k_half_heads", 1, (32768, 32768), (6, 6), (32, 4), 4096, "head_kv", "batched"),
        # many short chats of odd lengths and widths in one Cohort, history in the Cohort's natural packing
        _case("ragged_short_24", 24, (33, 3000), (1, 8), (32, 8), 1024, "token", "batched"),
        # one query per KV head (multi-head attention, no draft): plain decoding over resident history
        _case("decode_8x8k", 8, (8191, 8191), (1, 1), (8, 8), 4096, "head", "batched"),
        # a few users of the 48-head target at its widest verification
        _case("four_requests_16k_48_heads", 4, (16384, 16384), (8, 8), (48, 8), 4096, "head_kv", "batched"),
        # the benchmark round: 16 users at 32K, everything resident, one batched call
        _case("cohort_16x32k", 16, (32768, 32768), (6, 6), (32, 8), 4096, "head_kv", "batched"),
        # the same Cohort attended chunk by chunk as chunks become available
        _case("cohort_16x32k_by_chunk", 16, (32768, 32768), (6, 6), (32, 8), 4096, "token", "per_chunk"),
        # the 64-head target at its widest verification, 64 query rows on every KV head
        _case("cohort_16x32k_64_heads", 16, (32768, 32768), (8, 8), (64, 8), 4096, "head_kv", "batched"),
        # a full Cohort of mixed users: context lengths over a factor of 32, widths 1 to 8
        _case("ragged_64", 64, (2048, 65536), (1, 8), (32, 8), 4096, "head_kv", "batched"),
        # the largest round: 32 users at 128K with outlier keys
        _case("cohort_32x128k", 32, (131072, 131072), (8, 8), (32, 8), 8192, "head_kv", "batched", outlier_keys=True),
        # history in host memory: every chunk crosses the host link and is attended as it lands
        _case("streamed_16k", 1, (16384, 16384), (5, 5), (32, 8), 2048, "token", "streamed"),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        heads = rng.choice(HEADS)
        group = heads[0] // heads[1]
        requests = log_int(1, 64)
        hi = log_int(48, 131072)
        lo = hi if rng.random() < 0.4 else max(1, log_int(max(1, hi // 32), hi))
        chunk = rng.choice((1024, 2048, 4096, 8192, 1000, 3333))
        chunk = max(chunk, -(-hi // MAX_CALL_CHUNKS))
        cmax = rng.randint(1, min(8, 64 // group))
        cmin = cmax if rng.random() < 0.5 else rng.randint(1, cmax)
        calls = rng.choice(("batched", "batched", "batched", "per_chunk", "streamed"))
        c = _case("", requests, (lo, hi), (cmin, cmax), heads, chunk, rng.choice(sorted(LAYOUTS)), calls,
                  outlier_keys=rng.random() < 0.25, shape_seed=rng.randrange(1 << 30))
        del c["name"]
        if _history_bytes(c) <= (MOST_STREAMED_BYTES if calls == "streamed" else MOST_HISTORY_BYTES):
            return c


def _shape(case):
    """Per request: history tokens (log-uniform over the case's range) and candidates."""
    r = random.Random(case["shape_seed"])
    lo, hi = case["tokens_min"], case["tokens_max"]
    lens = [min(hi, max(lo, int(round(math.exp(r.uniform(math.log(lo), math.log(hi))))))) for _ in range(case["requests"])]
    cand = [r.randint(case["cand_min"], case["cand_max"]) for _ in range(case["requests"])]
    return lens, cand


def _history_bytes(case):
    return sum(_shape(case)[0]) * case["kv_heads"] * TOKEN_BYTES


def _inputs(case, seed):
    """Queries, candidates and history chunks in device memory, from the seed alone.

    Normal values; keys carry one scale in [0.5, 2] per head and channel, and with outlier_keys one key row in
    100 is 8 times larger.  A chunk is one tensor holding its K and its V in the case's layout, with views of both
    as [tokens, KV heads, d]."""
    lens, cand = _shape(case)
    hq, hkv, d = case["q_heads"], case["kv_heads"], HEAD_DIM
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape):
        return torch.randn(shape, generator=gen, device="cuda", dtype=torch.bfloat16)

    rows = sum(cand)
    scale = (torch.rand(hkv, d, generator=gen, device="cuda") * 1.5 + 0.5).to(torch.bfloat16)

    def keys(k):      # [tokens, KV heads, d], in place
        k *= scale
        if case["outlier_keys"]:
            k *= torch.where(torch.rand(k.shape[:2], generator=gen, device="cuda") < 0.01, 8.0, 1.0).to(k.dtype).unsqueeze(-1)

    q, kc, vc = normal(rows, hq, d), normal(rows, hkv, d), normal(rows, hkv, d)
    keys(kc)
    chunks, S = [], case["chunk_tokens"]
    for j in range(-(-max(lens) // S)):
        cl = [max(0, min(S, n - j * S)) for n in lens]
        t = sum(cl)
        if case["layout"] == "token":
            kv = normal(2, t, hkv, d)
            k, v = kv[0], kv[1]
        elif case["layout"] == "head":
            kv = normal(2, hkv, t, d)
            k, v = kv[0].transpose(0, 1), kv[1].transpose(0, 1)
        else:
            kv = normal(hkv, t, 2, d)
            k, v = kv[:, :, 0].transpose(0, 1), kv[:, :, 1].transpose(0, 1)
        keys(k)
        chunks.append((kv, k, v, cl))
    return q, kc, vc, chunks, lens, cand


class _Round:
    """What a serving loop holds between rounds: inputs, the descriptor, a zero-filled workspace, outputs."""

    def __init__(self, case, seed):
        q, kc, vc, chunks, _, cand = _inputs(case, seed)
        layout = LAYOUTS[case["layout"]]
        hq, hkv = case["q_heads"], case["kv_heads"]
        self.q, self.kc, self.vc, self.calls = q, kc, vc, case["calls"]
        self.desc = ss.make_desc(cand, hq, hkv, HEAD_DIM, max_chunk_tokens=max(sum(c[3]) for c in chunks),
                                 kv_layout=layout, counters_zeroed=1)
        self.ws_bytes = ss.ss_round_workspace_bytes(self.desc)
        self.ws = torch.zeros(self.ws_bytes, dtype=torch.uint8, device="cuda")
        self.out = torch.empty(sum(cand), hq, HEAD_DIM, device="cuda")
        self.lse = torch.empty(sum(cand), hq, device="cuda")
        self.lens = [c[3] for c in chunks]
        if self.calls == "streamed":
            self.host = [c[0].cpu().pin_memory() for c in chunks]
            self.slots = [torch.empty(max(256, max(h.numel() * 2 for h in self.host)), dtype=torch.uint8, device="cuda")
                          for _ in range(2)]
            self.copy_stream = torch.cuda.Stream()
            self.pipe = ss.ss_pipeline_create(self.slots[0].data_ptr(), self.slots[1].data_ptr(),
                                              self.slots[0].numel(), self.copy_stream.cuda_stream)
        else:
            self.chunks = [c[0] for c in chunks]
            self.k = [c[1].data_ptr() for c in chunks]
            self.v = [c[2].data_ptr() for c in chunks]

    def __del__(self):
        if getattr(self, "pipe", None):
            torch.cuda.synchronize()
            ss.ss_pipeline_destroy(self.pipe)
            self.pipe = None


def prepare(case, seed):
    ss.load()
    return _Round(case, seed)


def run(s):
    stream = torch.cuda.current_stream().cuda_stream
    r = ss.ss_round_init(s.desc, s.q.data_ptr(), s.ws.data_ptr(), s.ws_bytes, stream)
    try:
        if s.calls == "batched":
            ss.ss_attend_history_chunks(r, s.k, s.v, s.lens, None, None, stream)
        elif s.calls == "per_chunk":
            for k, v, n in zip(s.k, s.v, s.lens):
                ss.ss_attend_history_chunk(r, k, v, n, None, None, stream)
        else:
            for h, n in zip(s.host, s.lens):
                ss.ss_pipeline_attend_chunk(s.pipe, r, h.data_ptr(), n, stream)
        ss.ss_attend_local_candidates(r, s.kc.data_ptr(), s.vc.data_ptr(), stream)
        ss.ss_round_finalize(r, s.out.data_ptr(), s.lse.data_ptr(), stream)
    finally:
        ss.ss_round_destroy(r)
    return s.out, s.lse


def work(case):
    lens, cand = _shape(case)
    hq, hkv, d = case["q_heads"], case["kv_heads"], HEAD_DIM
    rows = sum(cand)
    nbytes = (sum(lens) + rows) * hkv * TOKEN_BYTES + rows * hq * (2 * d + 4 * d + 4)
    pairs = sum(n * c + c * (c + 1) // 2 for n, c in zip(lens, cand)) * hq
    return {"bytes": nbytes, "flops": pairs * 4 * d}


def tolerance(case):
    # float32 sums over softmax weights carried to 2^-16 for the product with V: 2e-6 to 3e-6 from float64
    return {"rel": 1e-5, "max": 1e-4}


def exact(case, seed):
    q, kc, vc, chunks, lens, cand = _inputs(case, seed)
    hq, hkv, d = case["q_heads"], case["kv_heads"], HEAD_DIM
    G, scale = hq // hkv, HEAD_DIM ** -0.5
    out = torch.empty(sum(cand), hq, d, dtype=torch.float64, device="cuda")
    lse = torch.empty(sum(cand), hq, dtype=torch.float64, device="cuda")
    starts = [[sum(c[3][:b]) for b in range(len(lens))] for c in chunks]
    row = 0
    for b, n in enumerate(cand):
        causal = torch.ones(n, n, dtype=torch.bool, device="cuda").tril()
        visible = torch.cat([torch.ones(n, lens[b], dtype=torch.bool, device="cuda"), causal], 1)
        parts = [(c[1][s[b]:s[b] + c[3][b]], c[2][s[b]:s[b] + c[3][b]]) for c, s in zip(chunks, starts) if c[3][b]]
        for g in range(hkv):
            k = torch.cat([p[0][:, g] for p in parts] + [kc[row:row + n, g]]).double()
            v = torch.cat([p[1][:, g] for p in parts] + [vc[row:row + n, g]]).double()
            x = q[row:row + n, g * G:(g + 1) * G].reshape(n * G, d).double() @ k.t() * scale
            x = x.masked_fill(~visible.repeat_interleave(G, 0), float("-inf"))
            l = torch.logsumexp(x, 1)
            out[row:row + n, g * G:(g + 1) * G] = (torch.exp(x - l[:, None]) @ v).view(n, G, d)
            lse[row:row + n, g * G:(g + 1) * G] = l.view(n, G)
        row += n
    return out, lse
