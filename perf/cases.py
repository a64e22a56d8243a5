"""Timed workloads of the MISA indexer, called as a serving or prefill loop calls it.

The shapes are those of the package's own configurations (workloads.WORKLOADS: the indexers of
DeepSeek-V3.2, 64 heads, and GLM-5, 32 heads, at prefix lengths up to 131072), of its tests (odd
lengths, ragged batches, paged caches, a few queries per sequence) and of its benchmark.  A case is
one indexer layer for one batch:

kind "step"   a decode step of a serving loop: the pooled keys of earlier tokens are kept, the block
              of the newest token is pooled again, then heads are routed, the cache is scored and
              the top-k taken (with k_cand > 0 also the dense re-rank).  graph: the step is captured
              once into a HIP graph and replayed, as bench.py does.
kind "pass"   Indexer.run: the whole pass including the pooling of the cache.
kind "score"  Indexer.score alone, on routed heads: the score matrix is the result.
kind "hisa"   the HISA comparison indexer (block scores, m best blocks, dense scores inside them).

All inputs are drawn on the GPU from the seed: Gaussian keys with a topic direction per segment of
2048 tokens and queries whose matching heads share it, gates of both signs, a few planted needle
keys, fp8 keys with one scale per token (the recipe of workloads.make_inputs, which draws on the
host and would be too slow here).
"""
from __future__ import annotations

import math

import torch

from paper_2605_07363_amd import misa

D = 128
KEY_BYTES = {"f32": 512, "bf16": 256, "e4m3": 132}   # one key row, with its scale for fp8
ELEM = {"f32": 4, "bf16": 2, "e4m3": 1}


def _case(name, kind, n_seq, L, n_q, H, h, B, k, k_dtype, q_dtype="bf16", k_cand=0, fused=False, page=0,
          ragged=False, graph=False, m=0):
    c = dict(kind=kind, n_seq=n_seq, L=L, n_q=n_q, H=H, h=h, B=B, k=k, k_dtype=k_dtype, q_dtype=q_dtype,
             k_cand=k_cand, fused=fused, page=page, ragged=ragged, graph=graph, m=m)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: one short fp32 sequence, one query (configuration c0); launches and host time count
        _case("decode_tiny_f32", "pass", 1, 4096, 1, 64, 8, 64, 256, "f32", "f32"),
        # interactive serving of one long conversation: batch 1, odd length, paged fp8 cache, captured step
        _case("decode_single_paged", "step", 1, 100003, 1, 64, 8, 64, 2048, "e4m3", page=64, graph=True),
        # batched serving, pooled keys maintained (configuration c1)
        _case("decode_batch_bf16", "step", 64, 32768, 1, 64, 8, 64, 2048, "bf16"),
        # long-context batch right after its prefill: the whole pass with pooling (configuration c3)
        _case("decode_long_fp8", "pass", 32, 131072, 1, 32, 8, 128, 2048, "e4m3"),
        # a few draft tokens per sequence verified together (multi-token decode)
        _case("decode_draft", "step", 16, 32768, 4, 64, 8, 64, 2048, "bf16"),
        # MISA-dagger decode on a ragged batch: 4 k candidates re-ranked by all heads
        _case("decode_rerank_ragged", "step", 16, 65536, 1, 64, 8, 128, 2048, "e4m3", k_cand=8192, ragged=True),
        # the tail of a prompt: a short chunk of odd size, whole pass, separate calls
        _case("prefill_short", "pass", 1, 10007, 333, 64, 8, 64, 2048, "bf16"),
        # a prefill chunk with the score matrix kept (configuration c2)
        _case("prefill_chunk", "pass", 1, 65536, 4096, 64, 8, 64, 2048, "bf16"),
        # MISA-dagger prefill, scoring and top-k fused (configuration c4)
        _case("prefill_dagger", "pass", 1, 131072, 2048, 64, 8, 64, 2048, "e4m3", k_cand=8192, fused=True),
        # the same with fp8 queries on the fp8 matrix instruction, two sequences, odd length
        _case("prefill_fp8_queries", "pass", 2, 50021, 1024, 64, 8, 64, 2048, "e4m3", "e4m3_matrix", 8192, True),
        # the scoring stage alone, 32-head indexer with 16 active heads, several sequences
        _case("prefill_score_h16", "score", 2, 32768, 1500, 32, 16, 128, 2048, "bf16"),
        # the HISA comparison indexer on a prefill chunk: 64 blocks of 128 tokens
        _case("hisa_prefill", "hisa", 1, 65536, 1024, 64, 8, 128, 2048, "bf16", m=64),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "pass", "pass", "pass", "score", "hisa"])
    H = rng.choice([32, 64])
    h = rng.choice([8, 8, 8, 4, 16])
    B = rng.choice([64, 128, 1024])
    k = rng.choice([512, 2048])
    k_dtype = rng.choice(["bf16", "e4m3"])
    if kind == "step" or (kind == "pass" and rng.random() < 0.3):
        L = _log(rng, 2048, 131072)
        n_seq = _log(rng, 1, max(1, min(64, (4 << 20) // L)))
        n_q = rng.choice([1, 1, 1, 2, 3, 5]) if kind == "step" else 1
        dagger = rng.random() < 0.3
        return _case(None, kind, n_seq, L, n_q, H, h, B, k, k_dtype, k_cand=4 * k if dagger else 0,
                     page=rng.choice([0, 0, 64, 256]), ragged=n_q == 1 and n_seq > 1 and rng.random() < 0.5,
                     graph=kind == "step" and rng.random() < 0.3)
    L = _log(rng, 4096, 131072)
    n_q = _log(rng, 32, min(4096, L, (128 << 20) // L))
    n_seq = rng.choice([1, 1, 2])
    if kind == "hisa":
        return _case(None, kind, 1, L, min(n_q, 1024), H, h, 128, k, k_dtype, m=32 if k == 512 else 64)
    if kind == "score":
        return _case(None, kind, n_seq, L, n_q, H, h, B, k, k_dtype)
    dagger = rng.random() < 0.5
    matrix = k_dtype == "e4m3" and rng.random() < 0.4
    return _case(None, kind, n_seq, L, n_q, H, h, B, k, k_dtype, "e4m3_matrix" if matrix else "bf16",
                 4 * k if dagger else 0, fused=rng.random() < 0.5, page=rng.choice([0, 0, 0, 64]))


# ---------------------------------------------------------------- inputs
def _lengths(c):
    """Tokens of each sequence: all L, or spread evenly over L/4 .. L."""
    n = c["n_seq"]
    return [int(c["L"] * (0.25 + 0.75 * (i + 1) / n)) if c["ragged"] else c["L"] for i in range(n)]


def _first_pos(c):
    return c["L"] - c["n_q"]


def _fp8(x):
    """Per row: scale max|x| / 448, codes of x / scale."""
    amax = x.abs().amax(dim=-1)
    scale = torch.where(amax > 0, amax / 448.0, torch.ones_like(amax))
    codes = (x / scale[..., None]).clamp_(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8)
    return codes, scale.contiguous()


def _inputs(c, seed):
    """Contiguous inputs: K, kscale (or None), Q, W on the GPU."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    kw = dict(generator=g, device="cuda")
    n_seq, L, n_q, H = c["n_seq"], c["L"], c["n_q"], c["H"]
    inv = D ** -0.5
    topics = torch.nn.functional.normalize(torch.randn(8, D, **kw), dim=-1)
    q = torch.randn(n_seq, n_q, H, D, **kw) * inv
    w = torch.randn(n_seq, n_q, H, **kw) * H ** -0.5
    run = torch.randint(0, 8, (n_seq, -(-n_q // 512)), **kw).repeat_interleave(512, dim=1)[:, :n_q]
    home = torch.arange(H, device="cuda") % 8
    q += 0.3145 * (home == run[..., None])[..., None] * topics[run][:, :, None, :]
    if c["q_dtype"] == "e4m3_matrix":
        codes, scale = _fp8(q)
        q, q_st, w = codes.view(torch.float8_e4m3fn).float(), codes, w * scale
    else:
        q_st = q if c["q_dtype"] == "f32" else q.to(torch.bfloat16)
        q = q_st.float()
    K, scales = [], []
    for s in range(n_seq):
        seg = torch.randint(0, 8, (-(-L // 2048),), **kw).repeat_interleave(2048)[:L]
        x = torch.randn(L, D, **kw) * inv + 0.5 * topics[seg]
        n_needles = min(256, L // 64)
        at = torch.randperm(L, **kw)[:n_needles]
        head = torch.argsort(w[s, -1], descending=True)[:4][torch.arange(n_needles, device="cuda") % 4]
        t = torch.randint(0, n_q, (n_needles,), **kw)
        x[at] = 4.0 * torch.nn.functional.normalize(q[s, t, head], dim=-1)
        if c["k_dtype"] == "e4m3":
            x, sc = _fp8(x)
            scales.append(sc)
        K.append(x.to(torch.bfloat16) if c["k_dtype"] == "bf16" else x)
    return torch.stack(K), torch.stack(scales) if scales else None, q_st.contiguous(), w.contiguous()


def _routed_heads(c, seed):
    """Ascending random head sets, for the cases that time the scoring stage alone."""
    g = torch.Generator(device="cuda").manual_seed(seed + 1)
    r = torch.rand(c["n_seq"], c["n_q"], c["H"], generator=g, device="cuda")
    return r.argsort(dim=-1)[..., :c["h"]].sort(dim=-1).values.to(torch.int32).contiguous()


class _State:
    pass


def prepare(case, seed):
    c = case
    s = _State()
    K, ks, Q, W = _inputs(c, seed)
    q_pos = None
    if c["n_q"] > 1:
        q_pos = torch.arange(_first_pos(c), c["L"], dtype=torch.int32, device="cuda")
    seq_len = torch.tensor(_lengths(c), dtype=torch.int32, device="cuda") if c["ragged"] else None
    q_code = {"f32": misa.F32, "bf16": misa.BF16, "e4m3_matrix": misa.FP8_E4M3_MATRIX}[c["q_dtype"]]
    p = misa.Problem(c["n_seq"], c["L"], c["n_q"], c["H"], c["B"], c["h"], misa.DTYPE_CODES[c["k_dtype"]], q_code,
                     q_pos, seq_len)
    dv = {"K": K, "kscale": ks, "problem": p}
    if c["page"]:
        dv = misa.paginate(dv, c["page"], seed=seed)
    s.case, s.K, s.ks, s.Q, s.W, s.p = c, dv["K"], dv["kscale"], Q, W, dv["problem"]
    if c["kind"] == "hisa":
        rows = (c["n_seq"], c["n_q"])
        s.Kp = torch.empty((c["n_seq"], p.M, D), dtype=torch.float32, device="cuda")
        misa.pool_keys(s.p, s.K, s.ks, s.Kp, misa.alloc_workspace(s.p, misa.OP_POOL))
        s.ws = misa.alloc_workspace(s.p, misa.OP_HISA, c["m"])
        s.blocks = torch.empty(rows + (c["m"],), dtype=torch.int32, device="cuda")
        s.idx = torch.empty(rows + (c["k"],), dtype=torch.int32, device="cuda")
        s.val = torch.empty(rows + (c["k"],), dtype=torch.float32, device="cuda")
        return s
    s.ix = misa.Indexer(s.p, c["k"], c["k_cand"], want_E=True, fused=c["fused"])
    if c["kind"] == "score":
        s.ix.heads.copy_(_routed_heads(c, seed))
    if c["kind"] == "step":
        s.newest = torch.tensor(_lengths(c), dtype=torch.int32, device="cuda") - 1
        s.ix.pool(s.K, s.ks)          # the pooled keys a serving loop already holds
        s.graph = None
        if c["graph"]:
            side = torch.cuda.Stream()
            side.wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(side):
                _step(s)
            torch.cuda.current_stream().wait_stream(side)
            s.graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(s.graph):
                _step(s)
    return s


# ---------------------------------------------------------------- one pass
def _step(s):
    ix = s.ix
    ix.pool_update(s.K, s.ks, s.newest, 1)
    ix.route(s.Q, s.W, s.K, s.ks)
    ix.score(s.Q, s.W, s.K, s.ks)
    ix.select()
    if ix.k_cand:
        ix.refine(s.Q, s.W, s.K, s.ks)


def run(state):
    s = state
    kind = s.case["kind"]
    if kind == "hisa":
        misa.hisa_select(s.p, s.Q, s.W, s.Kp, s.K, s.ks, s.case["m"], s.case["k"], s.idx, s.val, s.blocks, s.ws)
        return {"blocks": s.blocks, "idx": s.idx, "val": s.val}
    ix = s.ix
    if kind == "score":
        ix.score(s.Q, s.W, s.K, s.ks)
        return {"S": ix.S}
    if kind == "step":
        if s.graph is not None:
            s.graph.replay()
        else:
            _step(s)
        return {"Kp": ix.Kp, "E": ix.E, "heads": ix.heads, "S": ix.S, "idx": ix.idx}
    ix.run(s.K, s.ks, s.Q, s.W)
    return {"Kp": ix.Kp, "E": ix.E, "heads": ix.heads, "idx": ix.idx}


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    c = case
    lens = _lengths(c)
    rows = c["n_seq"] * c["n_q"]
    kb = KEY_BYTES[c["k_dtype"]]
    keys = sum(lens) * kb                                            # the cache, read once
    pairs = sum(sum(min(n, _first_pos(c) + t + 1) if c["n_q"] > 1 else n for t in range(c["n_q"])) for n in lens)
    q_bytes = rows * c["H"] * (D * ELEM["e4m3" if c["q_dtype"] == "e4m3_matrix" else c["q_dtype"]] + 4)
    blocks = pairs / c["B"]                                          # (query, visible block) pairs
    out_k = rows * c["k"] * (8 if c["kind"] == "hisa" else 4)        # indices (HISA: and values)
    if c["kind"] == "score":
        return {"bytes": keys + q_bytes + rows * c["h"] * 4 + rows * c["L"] * 4, "flops": 2.0 * D * c["h"] * pairs}
    kp = sum(-(-n // c["B"]) for n in lens) * D * 4
    if c["kind"] == "hisa":
        cand = rows * min(c["m"] * c["B"], c["L"])
        return {"bytes": keys + kp + q_bytes + out_k + rows * c["m"] * 4,
                "flops": 2.0 * D * c["H"] * (blocks + cand)}
    flops = 2.0 * D * (c["H"] * blocks + c["h"] * pairs)
    if c["k_cand"]:
        flops += 2.0 * D * c["H"] * sum(min(c["k_cand"], n) for n in lens) * c["n_q"]
    step = c["kind"] == "step"
    b = keys + kp + q_bytes + out_k + rows * (c["H"] + c["h"]) * 4
    if step:
        b += rows * c["L"] * 4                                       # the score matrix is one of its results
    return {"bytes": b, "flops": flops + (0 if step else sum(lens) * D)}


# Relative error measured against exact() on the listed and some drawn cases: score matrices
# 6e-8 .. 9e-8, pooled keys up to 9e-8, router scores E 6e-8 .. 1.1e-6 (the router carries pooled
# keys as two bf16 pieces; largest for blocks of 1024 tokens).  Four times that is stated.  A change
# of rounding can swap two near-tied entries at the edge of a top-k, which moves the ascending
# positions between them: a row in some thousands, allowed for in "differ" (and, for the values that
# the HISA call reports at those positions, in "rel" and "max").
def tolerance(case):
    if case["kind"] == "score":
        return {"rel": 4e-7, "max": 1e-4}
    if case["kind"] == "hisa":
        return {"rel": 0.01, "max": 1.0 - 1e-6, "differ": 0.01}
    return {"rel": 5e-6, "max": 2e-4, "differ": 0.01}


# ---------------------------------------------------------------- 64-bit reference
def _keys64(c, K, ks, s):
    if c["k_dtype"] == "e4m3":
        return K[s].view(torch.float8_e4m3fn).float().double() * ks[s].double()[:, None]
    return K[s].double()


def _visible(c, s):
    n = _lengths(c)[s]
    if c["n_q"] == 1:
        return torch.tensor([n], device="cuda")
    return (torch.arange(_first_pos(c), c["L"], device="cuda") + 1).clamp(max=n)


def _route64(c, q, w, k, n):
    """E [n_q, H] of one sequence: complete blocks of each query's prefix and the mean of its tail."""
    B = c["B"]
    csum = torch.cat([torch.zeros(1, D, dtype=torch.float64, device="cuda"), k.cumsum(0)])
    nb = c["L"] // B
    kp = (csum[B:nb * B + 1:B] - csum[:(nb - 1) * B + 1:B]) / B if nb else csum[:0]
    full, rest = n // B, n % B
    tail = (csum[n] - csum[full * B]) / rest.clamp(min=1)[:, None]
    step = max(1, (1 << 26) // (c["H"] * max(nb, 1)))
    out = []
    for a in range(0, q.shape[0], step):
        e = slice(a, a + step)
        dots = (q[e].reshape(-1, D) @ kp.T).relu_().view(q[e].shape[0], c["H"], nb)
        dots *= torch.arange(nb, device="cuda") < full[e][:, None, None]
        t = torch.matmul(q[e], tail[e][:, :, None]).squeeze(-1).relu()
        total = dots.sum(-1) + t * (rest[e] > 0)[:, None]
        out.append(w[e].abs() * total / (full[e] + (rest[e] > 0)).clamp(min=1)[:, None])
    return torch.cat(out), kp


def _score64(c, q, w, k, n, heads):
    """S [n_q, L] with the listed heads; -inf where a key is not visible."""
    S = torch.full((q.shape[0], c["L"]), -math.inf, dtype=torch.float64, device="cuda")
    step = max(1, (1 << 27) // (heads.shape[-1] * c["L"]))
    pos = torch.arange(c["L"], device="cuda")
    for a in range(0, q.shape[0], step):
        e = slice(a, a + step)
        hd = heads[e].long()
        qh = torch.gather(q[e], 1, hd[..., None].expand(-1, -1, D))
        wh = torch.gather(w[e], 1, hd)
        dots = (qh.reshape(-1, D) @ k.T).relu_().view(hd.shape[0], hd.shape[1], c["L"])
        dots *= wh[..., None]
        S[e] = torch.where(pos < n[e][:, None], dots.sum(1), S[e])
    return S


def exact(case, seed):
    """Pooled keys, router scores and, where the call leaves them, token scores; index outputs and
    the values at them have no 64-bit counterpart (a near-tie moves whole positions)."""
    c = case
    K, ks, Q, W = _inputs(c, seed)
    if c["q_dtype"] == "e4m3_matrix":
        Q = Q.view(torch.float8_e4m3fn).float()
    if c["kind"] == "hisa":
        return None
    E, S, Kp = [], [], []
    heads = _routed_heads(c, seed) if c["kind"] == "score" else None
    for s in range(c["n_seq"]):
        k, n = _keys64(c, K, ks, s), _visible(c, s)
        q, w = Q[s].double(), W[s].double()
        if c["kind"] == "score":
            S.append(_score64(c, q, w, k, n, heads[s]))
            continue
        length = _lengths(c)[s]
        e, _ = _route64(c, q, w, k, n)
        E.append(e)
        M, B = -(-c["L"] // c["B"]), c["B"]
        csum = torch.cat([torch.zeros(1, D, dtype=torch.float64, device="cuda"), k.cumsum(0)])
        lo = (torch.arange(M, device="cuda") * B).clamp(max=length)
        hi = (lo + B).clamp(max=length)
        Kp.append((csum[hi] - csum[lo]) / (hi - lo).clamp(min=1)[:, None])
        if c["kind"] == "step":
            top = torch.topk(e, c["h"], dim=-1).indices.sort(dim=-1).values
            S.append(_score64(c, q, w, k, n, top))
    if c["kind"] == "score":
        return {"S": torch.stack(S)}
    out = {"Kp": torch.stack(Kp), "E": torch.stack(E), "heads": None, "idx": None}
    if c["kind"] == "step":
        out["S"] = torch.stack(S)
    return out
