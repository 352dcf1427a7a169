"""Timed cases of the routed attention library: what its users call, over the sizes they call it at.

A case is a dict of plain values with a ``kind``:

  prefill   tilemix_prefill (quantize-once operands), or tilemix_prefill_fused with fused = True
  varlen    tilemix_prefill_varlen over a packed batch of sequences of different lengths
  decode    tilemix_decode, one token per sequence against an INT8 key/value cache; with
            ragged = True each sequence has its own cache length
  cache     tilemix_quantize_kv, building the INT8 key/value cache of a batch

``listed`` holds the named cases, ``draw`` makes one more of the same ranges, ``prepare`` makes the
device tensors of a case from a seed, ``run`` is one call, ``exact`` the same result in float64
with plain torch, ``work`` the bytes and operations the call cannot do without, and ``tolerance``
the error another correct implementation of the same precision may show.
"""

from __future__ import annotations

import math

import numpy as np
import torch

import paper_2608_17336_amd as tm

BLOCK_N = 64     # keys per routed tile, and per key scale block
BLOCK_Q = 128    # query rows per scale block


def _cdiv(a, b):
    return -(-a // b)


# ------------------------------------------------------------------------------------ cases

def listed():
    return [
        # The smallest prefill: a short prompt of a small multi-head model.  Launches and latency.
        dict(name="prefill-1k-mha-d64", kind="prefill", B=1, Hq=2, Hk=2, d=64, Lq=1024, Lk=1024,
             bm=64, g=1, mask="bernoulli", rho=0.5, causal=True, outliers=False, fused=False),
        # An ordinary prompt of a grouped-query model, half its tile groups on each route.
        dict(name="prefill-8k-gqa", kind="prefill", B=1, Hq=32, Hk=8, d=128, Lq=8192, Lk=8192,
             bm=128, g=1, mask="bernoulli", rho=0.5, causal=True, outliers=True, fused=False),
        # The headline workload: 32K tokens, three quarters of the groups on the INT8 route.
        dict(name="prefill-32k-gqa", kind="prefill", B=1, Hq=32, Hk=8, d=128, Lq=32768, Lk=32768,
             bm=128, g=4, mask="bernoulli", rho=0.75, causal=True, outliers=True, fused=False),
        # A long document: FP16 at the sink and near the diagonal, INT8 elsewhere.
        dict(name="prefill-128k-gqa", kind="prefill", B=1, Hq=32, Hk=8, d=128, Lq=131072, Lk=131072,
             bm=128, g=16, mask="sinkband", rho=0.0, causal=True, outliers=True, fused=False),
        # The largest: a batch of four 64K sequences with every tile on the FP16 route (exact
        # attention through the same kernel, which the caller announces with route_hint 0).
        dict(name="prefill-64k-b4-fp16", kind="prefill", B=4, Hq=64, Hk=8, d=128, Lq=65536, Lk=65536,
             bm=128, g=8, mask="zero", rho=0.0, causal=True, outliers=False, fused=False),
        # One chunk of a chunked prefill: few new query rows against a longer, ragged cache.
        dict(name="prefill-chunk-ragged", kind="prefill", B=2, Hq=16, Hk=4, d=128, Lq=500, Lk=9777,
             bm=128, g=2, mask="one", rho=1.0, causal=True, outliers=True, fused=False),
        # The fused on-the-fly operand mode (no K8 in memory) at an ordinary length.
        dict(name="prefill-8k-fused", kind="prefill", B=1, Hq=32, Hk=8, d=128, Lq=8192, Lk=8192,
             bm=128, g=1, mask="bernoulli", rho=0.5, causal=True, outliers=True, fused=True),
        # A packed batch of prompts from one token to 8K.
        dict(name="varlen-9-prompts", kind="varlen", Hq=32, Hk=8, d=128, bm=128, g=4,
             lens="8192,6000,4096,3001,2048,1024,512,123,1", mask="bernoulli", rho=0.75,
             causal=True, outliers=True),
        # One decode step of a single chat of 4K tokens: latency.
        dict(name="decode-4k", kind="decode", B=1, Hq=32, Hk=8, d=128, Lk=4096, g=1,
             mask="bernoulli", rho=0.5, ragged=False, outliers=True),
        # One decode step of a serving batch whose sequences have different lengths.
        dict(name="decode-ragged-b32", kind="decode", B=32, Hq=32, Hk=8, d=128, Lk=8192, g=2,
             mask="one", rho=1.0, ragged=True, outliers=True),
        # One decode step of four 64K sequences: memory bandwidth.
        dict(name="decode-64k-b4", kind="decode", B=4, Hq=64, Hk=8, d=128, Lk=65536, g=8,
             mask="bernoulli", rho=0.5, ragged=False, outliers=False),
        # Building the INT8 cache of a batch after its prefill.
        dict(name="cache-16k-b2", kind="cache", B=2, Hk=8, d=128, Lk=16384, outliers=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# Largest drawn prefill, in legal pairs x heads: below the 64K batch of four.
_MAX_PAIRS = 1.5e11


def draw(rng):
    kind = rng.choice(["prefill", "prefill", "prefill", "varlen", "decode", "decode", "cache"])
    Hq, Hk = rng.choice([(2, 2), (8, 8), (8, 2), (16, 4), (28, 4), (32, 8), (32, 8), (64, 8)])
    d = rng.choice([64, 128, 128])
    outliers = rng.random() < 0.5
    if kind == "cache":
        B = rng.choice([1, 2, 4, 8])
        return dict(kind=kind, B=B, Hk=Hk, d=d, Lk=_log_int(rng, 200, 65536 // B), outliers=outliers)
    mask, rho = rng.choice([("bernoulli", 0.5), ("bernoulli", 0.75), ("one", 1.0), ("zero", 0.0),
                            ("band", 0.75), ("bigbird", 0.5)])
    if kind == "decode":
        B = rng.choice([1, 2, 4, 8, 16, 32])
        if mask in ("band", "bigbird"):
            mask, rho = "bernoulli", rho
        return dict(kind=kind, B=B, Hq=Hq, Hk=Hk, d=d, Lk=_log_int(rng, 100, min(131072, 262144 // B)),
                    g=rng.choice([1, 2, 4, 8]), mask=mask, rho=rho, ragged=rng.random() < 0.5,
                    outliers=outliers)
    bm = rng.choice([64, 128, 128])
    if kind == "varlen":
        lens = [_log_int(rng, 1, 8192) for _ in range(rng.randint(2, 12))]
        return dict(kind=kind, Hq=Hq, Hk=Hk, d=d, bm=bm, g=rng.choice([1, 2, 4]),
                    lens=",".join(str(x) for x in lens), mask="zero" if mask == "zero" else "bernoulli",
                    rho=rho, causal=True, outliers=outliers)
    while True:
        B = rng.choice([1, 1, 2, 4])
        Lk = _log_int(rng, 100, 65536)
        Lq = Lk if rng.random() < 0.7 else _log_int(rng, 33, Lk)
        causal = rng.random() < 0.85
        if B * Hq * Lq * Lk <= _MAX_PAIRS:
            break
    g = tm.tilemix_auto_group_size(Lk) if rng.random() < 0.3 else rng.choice([1, 2, 4])
    return dict(kind="prefill", B=B, Hq=Hq, Hk=Hk, d=d, Lq=Lq, Lk=Lk, bm=bm, g=g, mask=mask, rho=rho,
                causal=causal, outliers=outliers, fused=rng.random() < 0.25)


# ----------------------------------------------------------------------------------- inputs

def _generator(seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed) * 7919 + 17)
    return gen


def _normal(gen, shape):
    out = torch.empty(shape, dtype=torch.float16, device="cuda")
    for part in out.split(8192, dim=1) if len(shape) == 4 else (out,):
        part.copy_(torch.randn(part.shape, generator=gen, device="cuda", dtype=torch.float32))
    return out


def _keys(gen, shape, outliers):
    """N(0, 1) keys; with outliers, 1% of each head's channels (at least one) are 8 times larger."""
    K = _normal(gen, shape)
    if outliers:
        H, d = shape[-2:]
        ch = torch.rand((H, d), generator=gen, device="cuda").argsort(-1)[:, :_cdiv(d, 100)]
        gain = torch.ones((H, d), dtype=torch.float16, device="cuda").scatter_(1, ch, 8.0)
        K *= gain
    return K


def _bernoulli_words(gen, rows, T_mask, W, rho):
    """Packed routing words [*rows, W] with i.i.d. INT8 bits of probability rho."""
    bits = torch.rand((*rows, W * 64), generator=gen, device="cuda") < rho
    bits[..., T_mask:] = False
    shift = torch.arange(64, device="cuda", dtype=torch.int64)
    return (bits.view(*rows, W, 64).to(torch.int64) << shift).sum(-1)


def _template_words(case, p, seed):
    kind = case["mask"]
    if kind == "sinkband":   # the first key group, and 4096 tokens next to the diagonal
        t = tm.Template("bigbird", band_w=_cdiv(4096, case["g"] * BLOCK_N), global_groups=1)
    elif kind in ("one", "zero"):
        t = tm.Template(kind)
    else:
        t = tm.tilemix_fit_template(p, tm.Template(kind, seed=int(seed)), case["rho"])
    return torch.from_numpy(tm.tilemix_route_template(p, t).view(np.int64)).cuda()


def _lens(case):
    return [int(x) for x in case["lens"].split(",")]


def prepare(case, seed):
    gen = _generator(seed)
    kind = case["kind"]
    if kind == "cache":
        shape = (case["B"], case["Lk"], case["Hk"], case["d"])
        return dict(kind=kind, K=_keys(gen, shape, case["outliers"]), V=_normal(gen, shape))
    Hq, Hk, d, g = case["Hq"], case["Hk"], case["d"], case["g"]
    scale = 1.0 / math.sqrt(d)
    hint = 0 if case["mask"] == "zero" else -1
    if kind == "varlen":
        lens = _lens(case)
        total, longest = sum(lens), max(lens)
        p = tm.Params(len(lens), Hq, Hk, longest, longest, d, case["bm"], BLOCK_N, g, case["causal"],
                      scale, False, hint)
        T_mask = _cdiv(_cdiv(longest, BLOCK_N), g)
        rows = sum(_cdiv(x, case["bm"]) for x in lens)
        cu = torch.tensor([0] + list(np.cumsum(lens)), dtype=torch.int32, device="cuda")
        return dict(kind=kind, Q=_normal(gen, (total, Hq, d)), K=_keys(gen, (total, Hk, d), case["outliers"]),
                    V=_normal(gen, (total, Hk, d)), cu=cu, longest=longest,
                    words=_bernoulli_words(gen, (rows, Hk), T_mask, _cdiv(T_mask, 64), case["rho"]),
                    O=torch.empty((total, Hq, d), dtype=torch.float16, device="cuda"),
                    ws=torch.empty(tm.tilemix_varlen_workspace_size(p, total, total), dtype=torch.uint8,
                                   device="cuda"),
                    args=dict(group_size=g, tile=(case["bm"], BLOCK_N), causal=case["causal"], scale=scale,
                              route_hint=hint))
    B, Lk = case["B"], case["Lk"]
    T_mask = _cdiv(_cdiv(Lk, BLOCK_N), g)
    W = _cdiv(T_mask, 64)
    kv = (B, Lk, Hk, d)
    if kind == "decode":
        p = tm.Params(B, Hq, Hk, 1, Lk, d, 128, BLOCK_N, g, True, scale, False, hint)
        K, V = _keys(gen, kv, case["outliers"]), _normal(gen, kv)
        K8, dK, V8, dV = tm.tilemix_quantize_kv(K, V)
        lens = None
        if case["ragged"]:   # from a short chat to a full cache, spread over their logarithm
            u = torch.rand((B,), generator=gen, device="cuda")
            lens = torch.exp(u * math.log(Lk / min(64, Lk)) + math.log(min(64, Lk))).round()
            lens = lens.clamp(1, Lk).to(torch.int32)
        if case["mask"] in ("one", "zero"):
            words = torch.full((1, Hk, 1, W), -1 if case["mask"] == "one" else 0, dtype=torch.int64,
                               device="cuda")
        else:
            words = _bernoulli_words(gen, (1, Hk, 1), T_mask, W, case["rho"])
        # A program that decodes from the cache keeps V8 only; V is held here for exact().
        Q = _normal(gen, (B, 1, Hq, d))
        return dict(kind=kind, Q=Q, K=K, V=V, cache=(K8, dK, V8, dV), words=words, lens=lens,
                    O=torch.empty_like(Q),
                    ws=torch.empty(tm.tilemix_decode_workspace_size(p), dtype=torch.uint8, device="cuda"),
                    args=dict(group_size=g, scale=scale, route_hint=hint))
    Lq = case["Lq"]
    p = tm.Params(B, Hq, Hk, Lq, Lk, d, case["bm"], BLOCK_N, g, case["causal"], scale, False, hint)
    if case["mask"] == "bernoulli":
        words = _bernoulli_words(gen, (1, Hk, _cdiv(Lq, case["bm"])), T_mask, W, case["rho"])
    else:
        words = _template_words(case, p, seed)
    size = tm.tilemix_fused_workspace_size if case["fused"] else tm.tilemix_workspace_size
    Q = _normal(gen, (B, Lq, Hq, d))
    return dict(kind=kind, fused=case["fused"], Q=Q, K=_keys(gen, kv, case["outliers"]), V=_normal(gen, kv),
                words=words, O=torch.empty_like(Q), ws=torch.empty(size(p), dtype=torch.uint8, device="cuda"),
                args=dict(group_size=g, tile=(case["bm"], BLOCK_N), causal=case["causal"], scale=scale,
                          route_hint=hint))


# -------------------------------------------------------------------------------------- run

def run(state):
    s = state
    kind = s["kind"]
    if kind == "cache":
        return tm.tilemix_quantize_kv(s["K"], s["V"])
    if kind == "varlen":
        return tm.tilemix_prefill_varlen(s["Q"], s["K"], s["V"], s["cu"], s["cu"], s["longest"],
                                         s["longest"], s["words"], O=s["O"], workspace=s["ws"], **s["args"])
    if kind == "decode":
        return tm.tilemix_decode(s["Q"], s["K"], *s["cache"], s["words"], O=s["O"], workspace=s["ws"],
                                 seqlens_k=s["lens"], **s["args"])
    call = tm.tilemix_prefill_fused if s["fused"] else tm.tilemix_prefill
    return call(s["Q"], s["K"], s["V"], s["words"], O=s["O"], workspace=s["ws"], **s["args"])


# ------------------------------------------------------------------------------------- work

def _legal_pairs(Lq, Lk, causal):
    if not causal:
        return Lq * Lk
    off = Lk - Lq
    return int(np.clip(np.arange(Lq, dtype=np.int64) + off + 1, 0, Lk).sum())


def work(case):
    """Every input read once and every output written once; 4 d operations per legal (query, key)
    pair of each query head (Q K^T and P V)."""
    kind, d = case["kind"], case["d"]
    if kind == "cache":
        n = case["B"] * case["Lk"] * case["Hk"]
        blocks = case["B"] * case["Hk"] * _cdiv(case["Lk"], BLOCK_N)
        return {"bytes": n * d * 2 * 3 + blocks * 2 * 2, "flops": n * d * 2 * 2}
    Hq, Hk, g = case["Hq"], case["Hk"], case["g"]
    if kind == "varlen":
        lens = _lens(case)
        pairs = sum(_legal_pairs(x, x, case["causal"]) for x in lens)
        rows = sum(_cdiv(x, case["bm"]) for x in lens)
        W = _cdiv(_cdiv(_cdiv(max(lens), BLOCK_N), g), 64)
        return {"bytes": sum(lens) * d * 4 * (Hq + Hk) + rows * Hk * W * 8, "flops": 4 * d * Hq * pairs}
    B, Lk = case["B"], case["Lk"]
    W = _cdiv(_cdiv(_cdiv(Lk, BLOCK_N), g), 64)
    if kind == "decode":
        keys = B * Lk
        if case["ragged"]:   # mean of lengths spread over their logarithm
            lo = min(64, Lk)
            keys = B * ((Lk - lo) / math.log(Lk / lo) if Lk > lo else Lk)
        rho = case["rho"]
        per_key = Hk * (d * rho + 2 * d * (1 - rho) + d + 4 / BLOCK_N)
        return {"bytes": keys * per_key + B * Hq * d * 4 + Hk * W * 8, "flops": 4 * d * Hq * keys}
    Lq = case["Lq"]
    pairs = B * Hq * _legal_pairs(Lq, Lk, case["causal"])
    words = Hk * _cdiv(Lq, case["bm"]) * W
    return {"bytes": B * d * 4 * (Lq * Hq + Lk * Hk) + words * 8, "flops": 4 * d * pairs}


def tolerance(case):
    """Cache: codes and scales are whole numbers and FP16 values fixed by the rule.  Attention: P is
    rounded to FP16 for P V (2^-12 relative, averaged over the keys) and O is rounded to FP16.
    Against exact(), the listed and 14 drawn cases measured 2.1e-4 to 3.3e-4 in the norm and up to
    1.1e-2 of the root mean square at one value (long sequences: their first rows are large against
    the rest); these are about four times that."""
    if case["kind"] == "cache":
        return "exact"
    return {"rel": 1.2e-3, "max": 4e-2}


# ------------------------------------------------------------------------------------ exact

def _codes(x, block):
    """Blockwise symmetric INT8 codes (float64) and FP16-stored scales (float64) of rows x [L, d]:
    scale = absmax / 127 and x / scale in correctly rounded float32, codes half to even."""
    L, d = x.shape
    n = _cdiv(L, block)
    pad = torch.zeros((n * block, d), dtype=torch.float64, device=x.device)
    pad[:L] = x.double()
    pad = pad.view(n, block, d)
    s32 = (pad.abs().amax((1, 2)) / 127.0).float()
    q = (pad / s32.double().clamp_min(1e-300)[:, None, None]).float().round().clamp(-127, 127)
    q = torch.where(s32[:, None, None] > 0, q, torch.zeros_like(q))
    return q.double().view(n * block, d)[:L], s32.half().double()


def _bits(words, T_mask):
    """Routing words [..., W] to a boolean map [..., T_mask]."""
    shift = torch.arange(64, device=words.device, dtype=torch.int64)
    b = (words[..., None] >> shift) & 1
    return b.flatten(-2)[..., :T_mask].bool()


def _attend(Q, K, V, words, bm, g, causal, scale):
    """One sequence in float64: Q [Lq, Hq, d], K, V [Lk, Hk, d], words [Hk, T_m, W]."""
    Lq, Hq, d = Q.shape
    Lk, Hk = K.shape[:2]
    off = Lk - Lq
    O = torch.zeros((Lq, Hq, d), dtype=torch.float64, device=Q.device)
    dev = Q.device
    route = _bits(words, _cdiv(_cdiv(Lk, BLOCK_N), g))
    group_of_key = torch.arange(Lk, device=dev) // BLOCK_N // g
    for hk in range(Hk):
        k, v = K[:, hk].double(), V[:, hk].double()
        k8, sk = _codes(K[:, hk], BLOCK_N)
        k8 = k8 * sk.repeat_interleave(BLOCK_N)[:Lk, None]
        for hq in range(hk * (Hq // Hk), (hk + 1) * (Hq // Hk)):
            q = Q[:, hq].double()
            q8, sq = _codes(Q[:, hq], BLOCK_Q)
            q8 = q8 * sq.repeat_interleave(BLOCK_Q)[:Lq, None]
            step = max(bm, (1 << 26) // max(Lk, 1) // bm * bm)
            for r0 in range(0, Lq, step):
                r1 = min(Lq, r0 + step)
                n = min(Lk, r1 + off) if causal else Lk
                if n <= 0:
                    continue
                rows = torch.arange(r0, r1, device=dev)
                int8 = route[hk][:, group_of_key[:n]][rows // bm]
                s = torch.where(int8, q8[r0:r1] @ k8[:n].T, q[r0:r1] @ k[:n].T) * scale
                if causal:
                    s.masked_fill_(torch.arange(n, device=dev)[None] > rows[:, None] + off, -math.inf)
                dead = torch.isinf(s.amax(1))
                p = torch.softmax(s, 1)
                p[dead] = 0.0
                O[r0:r1, hq] = p @ v[:n]
    return O


def exact(case, seed):
    kind = case["kind"]
    s = prepare(case, seed)
    if kind == "cache":
        B, L, Hk, d = s["K"].shape
        n = _cdiv(L, BLOCK_N)
        K8 = torch.empty((B, L, Hk, d), dtype=torch.float64, device="cuda")
        V8 = torch.zeros((B, Hk, n, d, BLOCK_N), dtype=torch.float64, device="cuda")
        dK, dV = (torch.empty((B, n, Hk), dtype=torch.float64, device="cuda") for _ in range(2))
        for b in range(B):
            for h in range(Hk):
                K8[b, :, h], dK[b, :, h] = _codes(s["K"][b, :, h], BLOCK_N)
                v, dV[b, :, h] = _codes(s["V"][b, :, h], BLOCK_N)
                pad = torch.zeros((n * BLOCK_N, d), dtype=torch.float64, device="cuda")
                pad[:L] = v
                V8[b, h] = pad.view(n, BLOCK_N, d).transpose(1, 2)
        return K8, dK, V8, dV
    if work(case)["flops"] > 2e13:
        return None
    g, scale = case["g"], s["args"]["scale"]
    if kind == "varlen":
        out, at, row = [], 0, 0
        for L in _lens(case):
            rows = _cdiv(L, case["bm"])
            words = s["words"][row:row + rows].transpose(0, 1)
            out.append(_attend(s["Q"][at:at + L], s["K"][at:at + L], s["V"][at:at + L], words, case["bm"],
                               g, case["causal"], scale))
            at, row = at + L, row + rows
        return torch.cat(out)
    if kind == "decode":
        B, Lk, Hk, d = s["K"].shape
        O = torch.zeros(s["Q"].shape, dtype=torch.float64, device="cuda")
        lens = [Lk] * B if s["lens"] is None else s["lens"].tolist()
        for b in range(B):
            V = torch.empty((Lk, Hk, d), dtype=torch.float64, device="cuda")
            K = torch.empty((Lk, Hk, d), dtype=torch.float64, device="cuda")
            route = _bits(s["words"][0, :, 0], _cdiv(_cdiv(Lk, BLOCK_N), g))
            of_key = torch.arange(Lk, device="cuda") // BLOCK_N // g
            n, G = lens[b], case["Hq"] // Hk
            for hk in range(Hk):
                v8, sv = _codes(s["V"][b, :, hk], BLOCK_N)
                V = v8 * sv.repeat_interleave(BLOCK_N)[:Lk, None]
                k8, sk = _codes(s["K"][b, :, hk], BLOCK_N)
                k8 = k8 * sk.repeat_interleave(BLOCK_N)[:Lk, None]
                q = s["Q"][b, 0, hk * G:(hk + 1) * G]
                q8, sq = _codes(q, 1)
                int8 = route[hk][of_key]
                sc = torch.where(int8, (q8 * sq[:, None]) @ k8.T, q.double() @ s["K"][b, :, hk].double().T)
                O[b, 0, hk * G:(hk + 1) * G] = torch.softmax(sc[:, :n] * scale, 1) @ V[:n]
        return O
    return torch.stack([_attend(s["Q"][b], s["K"][b], s["V"][b], s["words"][0], case["bm"], g,
                                case["causal"], scale) for b in range(case["B"])])
