"""What is timed: the work that a user of this library has it do, through its public entry points.

Three paths.  "layer" is one pass of the head-adaptive sparse prefill over one attention layer (block
scores, per-head selection, block-sparse attention), the way bench.py and the README call it.  "mass"
and "recovery" are the two dense passes of the offline profile that budgets come from.  Shapes are those
of the benchmark configurations (workloads/synth.py), the head counts of the parity tests, and generic
serving sizes; inputs follow the recipe of workloads/synth.py, drawn on the GPU.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2603_10353_amd as S

DEV = "cuda:0"
D = 128
RHO = 4.0                      # length of a head's mean query direction
SPLIT_SLOTS = 2048             # what bench.py --split-slots uses: never limits the piece length


def _batch_lengths(n, lo, hi, seed):
    r = np.random.Generator(np.random.Philox(key=[seed, 1]))
    return ",".join(str(int(x)) for x in np.exp(r.uniform(math.log(lo), math.log(hi), size=n)))


def listed():
    def layer(name, lens, hq, hkv, block, budget, **more):
        c = dict(name=name, path="layer", lens=lens, q_heads=hq, kv_heads=hkv, block=block, budget=budget, dense=0,
                 budget_seed=1000, c_lo=0.25, c_hi=6.0, entry="plain", packed=False, lse=True, kv_map="", tokens="")
        c.update(more)
        return c

    return [
        # one short prompt inside a serving loop that neither allocates nor wants the denominators
        layer("short_prompt", "777", 32, 8, 128, "log:0.2:1", entry="static", lse=False),
        # benchmark configuration 0: plain multi-head attention, 2K tokens, 64-token blocks
        layer("mha_2k_b64", "2048", 8, 8, 64, "choice:2:4:8:16", budget_seed=0, c_lo=0.5, c_hi=4.0),
        # a prefill batch of many short requests, QKV as a fused projection leaves it (28/4 heads)
        layer("batch_of_48", _batch_lengths(48, 20, 2000, 48), 28, 4, 128, "log:0.2:1", packed=True, lse=False),
        # an ordinary prompt with a ragged end, fused QKV
        layer("prompt_8k", "8231", 32, 8, 128, "log:0.02:0.5", packed=True, lse=False),
        # benchmark configuration 1: 32K context
        layer("layer_32k", "32768", 32, 8, 128, "log:0.02:0.5"),
        # the same layer with the finer block size
        layer("layer_32k_b64", "32768", 32, 8, 64, "log:0.02:0.5"),
        # benchmark configuration 2, the headline: 128K context, four heads at full budget
        layer("layer_128k", "131072", 32, 8, 128, "log:0.01:0.3", dense=4, budget_seed=2000),
        # one device's heads of a 64-head layer at 64K (configuration 3)
        layer("share_64k", "65536", 8, 2, 128, "two:0.03:0.4:0.3", budget_seed=3000),
        # benchmark configuration 4: a batch of very unequal long sequences, budgets per sequence and head
        layer("varlen_8k_to_128k", "8192,24576,65536,131072", 32, 8, 128, "log:0.01:0.5", budget_seed=4000),
        # mid-length prompt with dense-like heads through the entry point that cuts long rows
        layer("split_16k", "16384", 32, 8, 128, "log:0.01:0.3", dense=4, budget_seed=2000, entry="split"),
        # the offline recovery profile of a 32K sample, per block pair ...
        layer("mass_32k", "32768", 32, 8, 128, "", path="mass"),
        # ... and per query token at the profiled budget of 4096 tokens
        layer("recovery_32k", "32768", 32, 8, 128, "", path="recovery", tokens="4096"),
    ]


def draw(rng):
    """One more case of the same ranges: any length, head counts of the tests, both block sizes, every entry point."""
    log = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    hq, hkv = rng.choice([(32, 8), (28, 4), (40, 8), (8, 8), (8, 2), (16, 4)])
    path = rng.choice(["layer"] * 6 + ["mass", "recovery"])
    c = dict(path=path, q_heads=hq, kv_heads=hkv, block=rng.choice([128, 128, 64]), dense=0,
             budget_seed=rng.randrange(1 << 20), c_lo=0.25, c_hi=6.0, entry="plain", packed=rng.random() < 0.4,
             lse=rng.random() < 0.6, kv_map="", tokens="", budget="")
    if path == "mass":
        c["lens"] = str(log(1000, 32768))
    elif path == "recovery":
        t = log(1000, 16384)
        c["lens"] = str(t)
        c["tokens"] = ",".join(str(max(1, int(t * rng.uniform(0.02, 0.4)))) for _ in range(rng.choice([1, 1, 2, 3])))
    else:
        c["budget"] = rng.choice(["log:0.01:0.3", "log:0.02:0.5", "log:0.05:0.5", "log:0.2:1", "two:0.03:0.4:0.3"])
        c["dense"] = rng.choice([0, 0, 0, 1, 2])
        c["entry"] = rng.choice(["plain", "plain", "static", "split"])
        if rng.random() < 0.35:
            n = rng.choice([2, 3, 4, 8, 16, 40])
            total = log(4000, 65536)
            cut = sorted(rng.random() for _ in range(n - 1))
            c["lens"] = ",".join(str(max(1, int(total * (b - a)))) for a, b in zip([0.0] + cut, cut + [1.0]))
        else:
            c["lens"] = str(log(200, 65536))
        if hq == 8 and hkv == 2 and rng.random() < 0.5:
            c["kv_map"] = ",".join(str(x) for x in sorted(rng.choice([[0, 0, 0, 1, 1, 1, 1, 1], [0, 1, 1, 1, 1, 1, 1, 1]])))
    return c


def _lens(case):
    return [int(x) for x in case["lens"].split(",")]


def _n_blocks(case):
    return [-(-n // case["block"]) for n in _lens(case)]


def _budgets(case):
    """Key blocks per (sequence, head): part of the layer's plan, so a function of the case alone."""
    rng = np.random.Generator(np.random.Philox(key=[case["budget_seed"], 7]))
    hq, nbs = case["q_heads"], _n_blocks(case)
    kind, *args = case["budget"].split(":")
    if kind == "choice":
        k = rng.choice(np.array([int(x) for x in args]), size=hq)
        return np.stack([np.clip(k, 2, max(nb, 2)) for nb in nbs]).astype(np.int32).reshape(-1)
    if kind == "log":
        f = np.exp(rng.uniform(math.log(float(args[0])), math.log(float(args[1])), size=len(nbs) * hq)).reshape(len(nbs), hq)
    else:                                        # two:a:b:p -- fraction b with probability p, else a
        f = np.where(rng.uniform(size=(len(nbs), hq)) < float(args[2]), float(args[1]), float(args[0]))
    if case["dense"]:
        heads = np.random.Generator(np.random.Philox(key=[case["budget_seed"], 8])).choice(hq, size=case["dense"], replace=False)
        f[:, heads] = 1.0
    return np.stack([np.clip(np.floor(f[s] * nb + 0.5), 2, max(nb, 2)) for s, nb in enumerate(nbs)]).astype(np.int32).reshape(-1)


def _kv_of(case):
    if case["kv_map"]:
        return [int(x) for x in case["kv_map"].split(",")]
    g = case["q_heads"] // case["kv_heads"]
    return [h // g for h in range(case["q_heads"])]


def _inputs(case, seed, q, k, v):
    """Fill Q, K, V: noise, a mean direction per query head, and for every head the keys of the first block
    and of two heavy blocks per sequence pulled towards that direction by the head's concentration."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    rng = np.random.default_rng(seed)
    lens, hq, hkv, blk, kv_of = _lens(case), case["q_heads"], case["kv_heads"], case["block"], _kv_of(case)
    dirs = np.empty((hq, D), np.float32)
    for g in range(hkv):
        heads = [h for h in range(hq) if kv_of[h] == g]
        if heads:
            dirs[heads] = RHO * np.linalg.qr(rng.standard_normal((D, len(heads))))[0].T
    conc = rng.uniform(case["c_lo"], case["c_hi"], size=hq)
    m = torch.from_numpy(dirs).to(DEV)
    pull = torch.from_numpy((dirs * conc[:, None]).astype(np.float32)).to(DEV)
    total, step = sum(lens), 16384
    for t in range(0, total, step):
        n = min(step, total - t)
        q[t:t + n] = torch.randn((n, hq, D), device=DEV, generator=gen) + m
        if v is not None:
            v[t:t + n] = torch.randn((n, hkv, D), device=DEV, generator=gen)
    kf = torch.randn((total, hkv, D), device=DEV, generator=gen)
    begin = 0
    for n in lens:
        nb = -(-n // blk)
        for h in range(hq):
            heavy = rng.choice(np.arange(1, nb - 1), size=2, replace=False) if nb >= 4 else []
            for b in [0, *heavy]:
                kf[begin + int(b) * blk:begin + min(n, (int(b) + 1) * blk), kv_of[h]] += pull[h]
        begin += n
    k.copy_(kf)


def prepare(case, seed):
    lens, hq, hkv, blk = _lens(case), case["q_heads"], case["kv_heads"], case["block"]
    total = sum(lens)
    layer = case["path"] == "layer"
    n_v = hkv if layer else 0
    if case["packed"]:                           # column slices of one [T, Hq + 2 Hkv, 128] buffer
        width = hq + hkv + n_v
        qkv = torch.empty((total, width, D), dtype=torch.bfloat16, device=DEV)
        q, k, v = qkv[:, :hq], qkv[:, hq:hq + hkv], qkv[:, hq + hkv:] if n_v else None
        strides = dict(q_stride_t=width * D, q_stride_h=D, kv_stride_t=width * D, kv_stride_h=D)
    else:
        q = torch.empty((total, hq, D), dtype=torch.bfloat16, device=DEV)
        k = torch.empty((total, hkv, D), dtype=torch.bfloat16, device=DEV)
        v = torch.empty_like(k) if n_v else None
        strides = {}
    _inputs(case, seed, q, k, v)
    p = S.Problem(np.concatenate([[0], np.cumsum(lens)]), hq, hkv, blk, D,
                  kv_head_of=_kv_of(case) if case["kv_map"] else None, **strides)
    st = dict(case=case, p=p, q=q, k=k, v=v)
    floats = int(S.shplb_score_layout(p)[-1])
    if case["path"] == "mass":
        st["mass"] = torch.zeros(floats, dtype=torch.float32, device=DEV)
        return st
    if case["path"] == "recovery":
        st["tokens"] = np.array([int(x) for x in case["tokens"].split(",")], np.int32)
        st["recovery"] = torch.zeros((st["tokens"].size, hq, total), dtype=torch.float32, device=DEV)
        return st
    st["budgets"] = _budgets(case)
    ptr = S.shplb_sel_row_ptr(p, st["budgets"])
    st["sel_ptr"] = torch.from_numpy(ptr).to(DEV)
    st["sel_idx"] = torch.zeros(int(ptr[-1]), dtype=torch.int32, device=DEV)
    st["scores"] = torch.zeros(floats, dtype=torch.float32, device=DEV)   # only j <= i is written
    n_ws = S.shplb_split_workspace_bytes(p, SPLIT_SLOTS) if case["entry"] == "split" else S.shplb_workspace_bytes(p)
    st["ws"] = torch.empty(n_ws, dtype=torch.uint8, device=DEV)
    # the output has the strides of Q
    out = torch.zeros((total, width if case["packed"] else hq, D), dtype=torch.bfloat16, device=DEV)
    st["out"] = out[:, :hq]
    st["lse"] = torch.zeros((hq, total), dtype=torch.float32, device=DEV) if case["lse"] else None
    return st


def run(st):
    case, p, q, k, v = st["case"], st["p"], st["q"], st["k"], st["v"]
    stream = torch.cuda.current_stream()
    if case["path"] == "mass":
        S.shplb_block_mass(p, q, k, st["mass"], stream)
        return st["mass"]
    if case["path"] == "recovery":
        S.shplb_token_recovery(p, q, k, st["tokens"], st["recovery"], stream)
        return st["recovery"]
    ptr, idx, out, lse, ws = st["sel_ptr"], st["sel_idx"], st["out"], st["lse"], st["ws"]
    S.shplb_block_scores(p, q, k, st["scores"], ws, stream)
    S.shplb_select_topk_per_head(p, st["scores"], st["budgets"], ptr, idx, stream)
    if case["entry"] == "static":
        S.shplb_sparse_attn_prefill_static(p, q, k, v, ptr, idx, out, lse, None, stream)
    elif case["entry"] == "split":
        S.shplb_sparse_attn_prefill_split(p, q, k, v, ptr, idx, out, lse, None, ws, SPLIT_SLOTS, stream)
    else:
        S.shplb_sparse_attn_prefill(p, q, k, v, ptr, idx, out, lse, None, ws, stream)
    got = dict(scores=st["scores"], sel_idx=idx, out=out)
    if lse is not None:
        got["lse"] = lse
    return got


def work(case):
    """Each input read once, each output written once; products of the unmasked (query, key) pairs."""
    lens, hq, hkv, blk = _lens(case), case["q_heads"], case["kv_heads"], case["block"]
    total, nbs = sum(lens), _n_blocks(case)
    tri = hq * sum(nb * (nb + 1) // 2 for nb in nbs)             # block pairs (i, j <= i)
    if case["path"] != "layer":
        pairs = hq * sum(n * (n + 1) // 2 for n in lens)
        outs = tri if case["path"] == "mass" else (case["tokens"].count(",") + 1) * hq * total
        return {"bytes": 2 * D * total * (hq + hkv) + 4 * outs, "flops": 2 * D * pairs}
    budgets = _budgets(case).reshape(len(lens), hq)
    pairs = blocks = 0
    for s, n in enumerate(lens):
        i = np.arange(nbs[s])
        valid = np.minimum(blk, n - i * blk)
        for h in range(hq):
            sel = np.minimum(min(max(int(budgets[s, h]), 2), nbs[s]), i + 1)
            pairs += int(((sel - 1) * valid * blk + valid * (valid + 1) // 2).sum())
            blocks += int(sel.sum())
    nbytes = 2 * D * total * (2 * hq + 2 * hkv) + 4 * tri + 4 * blocks + (4 * hq * total if case["lse"] else 0)
    return {"bytes": nbytes, "flops": 4 * D * pairs + 2 * D * tri}


def tolerance(case):
    # Measured against 64-bit evaluations.  Layer: outputs are off by 2.2e-3 (bf16 probabilities and results)
    # and at most 0.024 of their size, selections from 64-bit scores are the same up to near-ties.  Profile
    # passes: fp32 sums, off by 2e-7 to 4e-7, single values by up to 5e-6, at 3000 tokens; longer sums at 32K.
    if case["path"] == "layer":
        return {"rel": 9e-3, "max": 0.1, "differ": 1e-4}
    return {"rel": 1e-5, "max": 1e-4}
