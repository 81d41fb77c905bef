"""Performance cases: what a program that uses this library has it do, from one decode step to a 128K training pass.

Every case goes through the package's public entry points with inputs, outputs and workspaces already on the GPU,
as a serving or training loop keeps them.  Kinds:
  train           forward, then backward, of a [B, H, N, D] batch (one sparse or full layer of a training step)
  train_packed    the same over sequences of different lengths packed per head
  prefill         forward only; with "cache" the prompt's keys and values are then stored into the reduced cache
  prefill_packed  forward over requests of different lengths packed per head
  decode          one generated token per sequence: store its key and value, attend over the reduced cache
  paged           the same over a paged cache shared by sequences of different context lengths
"""
import math
import random

import numpy as np
import torch

import paper_2410_01485_amd as lg

DTYPES = {"bf16": torch.bfloat16, "fp32": torch.float32}


def _case(name, kind, B, Hq, Hkv, D, N, sink, window, block=1, stride=0, dtype="bf16", **more):
    return dict({"name": name, "kind": kind, "B": B, "Hq": Hq, "Hkv": Hkv, "D": D, "N": N, "sink": sink,
                 "window": window, "block": block, "stride": stride, "dtype": dtype}, **more)


def listed():
    return [
        # one user generating token by token: a single short context with grouped heads, nothing but latency
        _case("decode_one", "decode", 1, 32, 8, 128, 1500, 64, 2048),
        # the decode benchmark: 16 sequences, ring caches of 64 + 4096 slots out of a 131072-token context
        _case("decode_batch16", "decode", 16, 32, 32, 128, 131072, 64, 4096),
        # the paper's block-sparse cache (every 64th block retained) under 64 query / 8 key-value heads
        _case("decode_strided_gqa", "decode", 8, 64, 8, 128, 100003, 64, 2048, 64, 64),
        # a serving engine's step: 48 sequences of very different lengths in a paged cache
        _case("decode_paged", "paged", 48, 32, 8, 128, 32768, 64, 4096, page=64, shortest=20, mix=1),
        # a short ragged prompt at the small head dimension, its cache filled for the generation that follows
        _case("prefill_short_d64", "prefill", 2, 16, 16, 64, 1003, 64, 512, cache=True),
        # block-strided prefill: own block and two before it, the sink block, every 8th earlier block
        _case("prefill_strided_32k", "prefill", 1, 32, 32, 128, 32768, 64, 192, 64, 8, cache=False),
        # a serving batch of many short prompts, packed without padding
        _case("prefill_packed", "prefill_packed", 256, 32, 32, 128, 2048, 64, 4096, shortest=256, mix=2),
        # long-context prefill with grouped heads
        _case("prefill_gqa_128k", "prefill", 1, 64, 8, 128, 131072, 64, 4096, cache=False),
        # the length-extension training pass of one sparse layer
        _case("train_128k", "train", 1, 32, 32, 128, 131072, 64, 4096),
        # the paper's block-sparse setting in training, grouped heads, a ragged length
        _case("train_strided_gqa", "train", 1, 64, 8, 128, 16001, 64, 2048, 64, 64),
        # training on packed documents, most of them shorter than the window
        _case("train_packed", "train_packed", 24, 32, 8, 128, 8192, 64, 4096, shortest=200, mix=3),
        # the float32 path: gradients of a small layer
        _case("train_fp32", "train", 2, 8, 4, 64, 1024, 16, 128, dtype="fp32"),
    ]


# Limits of a drawn case, in operations and bytes of its work(): below the largest listed one.
MOST_FLOPS = {"bf16": 1.5e13, "fp32": 1.0e10}
MOST_BYTES = 3.0e9


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _pattern(rng, kind, N):
    """sink, window, block, stride: token-exact or 64-token blocks, with or without strided columns, or full."""
    what = rng.choice(["token", "token", "block", "strided", "full"] if kind in ("train", "prefill")
                      else ["token", "token", "block", "strided"])
    if what == "token":
        return rng.choice([0, 4, 16, 64]), _log_int(rng, 100, 4096), 1, 0
    if what == "full":
        return 0, N, 1, 0
    return 64, 64 * _log_int(rng, 2, 64), 64, rng.choice([4, 8, 16, 64]) if what == "strided" else 0


def draw(rng):
    kind = rng.choice(["train", "train_packed", "prefill", "prefill_packed", "decode", "decode", "paged"])
    dtype = "fp32" if kind in ("train", "prefill", "decode") and rng.random() < 0.2 else "bf16"
    D = 64 if rng.random() < 0.3 else 128
    Hkv = rng.choice([1, 2, 4, 8, 16, 32])
    Hq = Hkv * rng.choice([1, 1, 2, 4, 8])
    more = {}
    if kind in ("train", "prefill"):
        B = rng.choice([1, 1, 2, 4])
        N = _log_int(rng, 64, 8192) if dtype == "fp32" else _log_int(rng, 300, 131072)
        if kind == "prefill":
            more = {"cache": rng.random() < 0.5}
    elif kind in ("train_packed", "prefill_packed"):
        B = _log_int(rng, 2, 256)
        N = _log_int(rng, 300, 32768)
        more = {"shortest": max(1, N // rng.choice([4, 16, 64])), "mix": rng.randrange(1 << 30)}
    else:
        B = _log_int(rng, 1, 64)
        N = _log_int(rng, 10, 131072)
        if kind == "paged":
            more = {"page": rng.choice([16, 32, 64, 128]), "shortest": max(1, N // rng.choice([2, 16, 256])),
                    "mix": rng.randrange(1 << 30)}
    sink, window, block, stride = _pattern(rng, kind, N)
    c = _case("", kind, B, Hq, Hkv, D, N, sink, window, block, stride, dtype, **more)
    del c["name"]
    c["Hq"] = min(c["Hq"], 64)
    c["Hkv"] = min(c["Hkv"], c["Hq"])
    while True:  # fewer heads, then fewer sequences, then a shorter context, until the case is within the limits
        w = work(c)
        if w["flops"] <= MOST_FLOPS[dtype] and w["bytes"] <= MOST_BYTES:
            return c
        if c["Hkv"] > 1:
            c["Hq"], c["Hkv"] = c["Hq"] // 2, c["Hkv"] // 2
        elif c["B"] > 1:
            c["B"] //= 2
        else:
            full = c["window"] >= c["N"] and block == 1
            c["N"] //= 2
            c["window"] = c["N"] if full else c["window"]
            if "shortest" in c:
                c["shortest"] = min(c["shortest"], c["N"])


def _lengths(case):
    """Lengths of the sequences of a packed or paged case: spread evenly over their logarithm, the longest is N."""
    rng = random.Random(case["mix"])
    return [case["N"]] + [_log_int(rng, case["shortest"], case["N"]) for _ in range(case["B"] - 1)]


def _row_keys(case, rows):
    """Live keys of the query rows (numpy array of positions)."""
    b = max(case["block"], 1)
    sb, wb, st = case["sink"] // b, case["window"] // b, case["stride"]
    qb = rows // b
    older = np.maximum(qb - wb + 1, 0)  # blocks older than the window
    below = np.minimum(qb, wb - 1) + np.minimum(sb, older)
    if st > 0:
        below = below + np.maximum(older // st - np.minimum(sb, older) // st, 0)
    return below * b + rows - qb * b + 1


def work(case):
    """Bytes: each input read once, each output written once.  Operations: 4 D per live pair forward, 10 D backward."""
    c = case
    e, D = (2 if c["dtype"] == "bf16" else 4), c["D"]
    if c["kind"] in ("decode", "paged"):
        lens = np.array(_lengths(c) if c["kind"] == "paged" else [c["N"]] * c["B"])
        keys = int(_row_keys(c, lens - 1).sum())
        new = 4.0 * c["B"] * c["Hkv"] * D * e  # the new rows of K and V, read and stored
        return {"bytes": 2.0 * keys * c["Hkv"] * D * e + new + c["B"] * c["Hq"] * (2.0 * D * e + 4),
                "flops": 4.0 * D * keys * c["Hq"]}
    lens = _lengths(c) if c["kind"].endswith("packed") else [c["N"]] * c["B"]
    rows = _row_keys(c, np.arange(max(lens)))
    upto = np.concatenate([[0], np.cumsum(rows)])
    pairs, T = float(sum(int(upto[n]) for n in lens)), float(sum(lens))
    q, kv, lse = T * c["Hq"] * D * e, T * c["Hkv"] * D * e, T * c["Hq"] * 4
    if c["kind"].startswith("train"):
        return {"bytes": 4 * q + 4 * kv + lse, "flops": 14.0 * D * pairs * c["Hq"]}
    cache = 0.0
    if c.get("cache"):
        slots = min(c["N"], c["sink"] + c["window"])
        cache = 2.0 * c["B"] * c["Hkv"] * slots * D * e
    return {"bytes": 2 * q + 2 * kv + lse + cache, "flops": 4.0 * D * pairs * c["Hq"]}


def tolerance(case):
    return {"rel": 1e-2} if case["dtype"] == "bf16" else {"rel": 1e-5}


def prepare(case, seed):
    c = dict(case)
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    dt = DTYPES[c["dtype"]]
    code = lg.LG_BF16 if c["dtype"] == "bf16" else lg.LG_F32
    B, Hq, Hkv, N, D = c["B"], c["Hq"], c["Hkv"], c["N"], c["D"]
    pat = (c["sink"], c["window"], c["block"], c["stride"])

    def rnd(*shape):
        return torch.randn(*shape, generator=gen, device="cuda", dtype=dt)

    def new(*shape, dtype=dt):
        return torch.zeros(*shape, device="cuda", dtype=dtype)

    def workspace(nbytes):
        return new(max(int(nbytes), 16), dtype=torch.uint8)

    s = {"kind": c["kind"], "pattern": pat, "N": N, "cache": bool(c.get("cache"))}
    if c["kind"] == "decode":
        slots = lg.lg_kv_cache_slots(N, *pat)
        s.update(q=rnd(B, Hq, D), k=rnd(B, Hkv, 1, D), v=rnd(B, Hkv, 1, D), kc=rnd(B, Hkv, slots, D),
                 vc=rnd(B, Hkv, slots, D), out=new(B, Hq, D), lse=new(B, Hq, dtype=torch.float32),
                 ws=workspace(lg.decode_cache_workspace_bytes(B, Hq, Hkv, N, D, *pat, code)))
    elif c["kind"] == "paged":
        lens, page = _lengths(c), c["page"]
        per_seq = -(-lg.lg_kv_cache_slots(N, *pat) // page)
        order = torch.randperm(B * per_seq, generator=gen, device="cuda").to(torch.int32)
        n = torch.tensor(lens, dtype=torch.int32, device="cuda")
        s.update(q=rnd(B, Hq, D), k=rnd(B, Hkv, 1, D), v=rnd(B, Hkv, 1, D), kc=rnd(B * per_seq, Hkv, page, D),
                 vc=rnd(B * per_seq, Hkv, page, D), table=order.reshape(B, per_seq).contiguous(), lens=n,
                 pos=n - 1, out=new(B, Hq, D), lse=new(B, Hq, dtype=torch.float32),
                 ws=workspace(lg.decode_paged_workspace_bytes(B, Hq, Hkv, N, D, *pat, code)))
    else:
        packed = c["kind"].endswith("packed")
        if packed:
            s["cu"] = [0] + [int(x) for x in np.cumsum(_lengths(c))]
            lead, T = (), s["cu"][-1]
        else:
            lead, T = (B,), N
        s.update(q=rnd(*lead, Hq, T, D), k=rnd(*lead, Hkv, T, D), v=rnd(*lead, Hkv, T, D))
        s.update(out=new(*lead, Hq, T, D), lse=new(*lead, Hq, T, dtype=torch.float32))
        if c["kind"].startswith("train"):
            s["dout"] = rnd(*lead, Hq, T, D)
            s.update(dq=new(*lead, Hq, T, D), dk=new(*lead, Hkv, T, D), dv=new(*lead, Hkv, T, D))
            s["ws"] = workspace(lg.bwd_varlen_workspace_bytes(s["cu"], Hq, Hkv, D, *pat, code) if packed
                                else lg.bwd_workspace_bytes(B, Hq, Hkv, N, D, *pat, code))
        elif s["cache"]:
            slots = lg.lg_kv_cache_slots(N, *pat)
            s.update(kc=new(B, Hkv, slots, D), vc=new(B, Hkv, slots, D))
    return s


def run(s):
    pat = s["pattern"]
    if s["kind"] == "decode":
        lg.lg_kv_ring_append(s["k"], s["v"], s["kc"], s["vc"], s["N"] - 1, *pat)
        lg.lg_sparse_attn_decode_cache(s["q"], s["kc"], s["vc"], s["out"], s["lse"], s["ws"], s["N"], *pat)
        return s["out"], s["lse"], s["kc"], s["vc"]
    if s["kind"] == "paged":
        lg.lg_kv_paged_append(s["k"], s["v"], s["kc"], s["vc"], s["table"], s["pos"], s["N"], *pat)
        lg.lg_sparse_attn_decode_paged(s["q"], s["kc"], s["vc"], s["table"], s["lens"], s["out"], s["lse"], s["ws"],
                                       s["N"], *pat)
        return s["out"], s["lse"], s["kc"], s["vc"]
    if s["kind"].endswith("packed"):
        lg.lg_sparse_attn_fwd_varlen(s["q"], s["k"], s["v"], s["out"], s["lse"], s["cu"], *pat)
        if s["kind"] == "prefill_packed":
            return s["out"], s["lse"]
        lg.lg_sparse_attn_bwd_varlen(s["q"], s["k"], s["v"], s["out"], s["lse"], s["dout"], s["dq"], s["dk"], s["dv"],
                                     s["ws"], s["cu"], *pat)
        return s["out"], s["lse"], s["dq"], s["dk"], s["dv"]
    lg.lg_sparse_attn_fwd(s["q"], s["k"], s["v"], s["out"], s["lse"], *pat)
    if s["kind"] == "train":
        lg.lg_sparse_attn_bwd(s["q"], s["k"], s["v"], s["out"], s["lse"], s["dout"], s["dq"], s["dk"], s["dv"], s["ws"],
                              *pat)
        return s["out"], s["lse"], s["dq"], s["dk"], s["dv"]
    if s["cache"]:
        lg.lg_kv_ring_append(s["k"], s["v"], s["kc"], s["vc"], 0, *pat)
        return s["out"], s["lse"], s["kc"], s["vc"]
    return s["out"], s["lse"]
