"""The calls whose speed is measured, and how their results are checked.

A case is one call sequence of the library's Python entry points on a batch of
a given shape:

  qkv     cw.qkv_rope_append: projection, rotary embedding and KV append
  append  cw.kv_append
  attn    cw.suffix_prefill_attn
  split   cw.suffix_prefill_attn_split with its automatic split count
  fused   cw.suffix_prefill_append_attn
  layer   cw.qkv_rope_append, then attention on its queries (split when the
          batch has fewer tiles than the GPU has compute units)
  step    a serving step of cw.BatchRunner: schedule, plan, upload, fused call,
          release

A batch is either given by sizes ("batch" requests of about "suffix" new and
"prefix" cached tokens, spread around them when "spread" is true) or by a
retrieval trace ("trace": the pool's prefix matches give the lengths). Values
are N(0, 1) in bfloat16, weights N(0, 1 / hidden); physical blocks are a random
permutation of the pool.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2606_19667_amd import batch as B
from paper_2606_19667_amd import cw
from paper_2606_19667_amd import workload as W

BS = 16
ROPE_BASE = 500000.0
HEADS = {  # query heads, KV heads, head_dim, hidden
    "tiny": (4, 1, 64, 256),
    "d64": (16, 4, 64, 1024),
    "qwen7b": (28, 4, 128, 3584),
    "llama8b": (32, 8, 128, 4096),
    "llama70b": (64, 8, 128, 8192),
}


def listed():
    return [
        # The smallest batch the framework runs (its smoke test): launch latency.
        dict(name="tiny-fused", op="fused", heads="tiny", batch=1, prefix=64, suffix=32),
        # One request of a lightly loaded 8B server, three of five chunks cached:
        # the layer's projection, then its attention.
        dict(name="single-qkv", op="qkv", heads="llama8b", batch=1, prefix=832, suffix=576),
        dict(name="single-split", op="split", heads="llama8b", batch=1, prefix=832, suffix=576),
        # Every evidence chunk cached (what the ordering aims for): only the
        # 64-token questions of 16 requests are prefilled.
        dict(name="question-qkv", op="qkv", heads="llama8b", batch=16, prefix=1344, suffix=64),
        dict(name="question-split", op="split", heads="llama8b", batch=16, prefix=1344, suffix=64),
        # A whole layer of a 7B model with seven query heads per KV head and a
        # bias, on a ragged batch of odd lengths.
        dict(name="qwen7b-ragged-layer", op="layer", heads="qwen7b", batch=6, prefix=700, suffix=411, spread=True,
             bias=True),
        # The 16-request trace batch of the benchmark: the layer's kernels by
        # themselves, and the whole serving step.
        dict(name="trace-append", op="append", heads="llama8b", trace=True, batch=16),
        dict(name="trace-qkv", op="qkv", heads="llama8b", trace=True, batch=16),
        dict(name="trace-attn", op="attn", heads="llama8b", trace=True, batch=16),
        dict(name="trace-step", op="step", heads="llama8b", trace=True, batch=16),
        # Long prompts: ten chunks of 512 tokens with 60 % of the blocks cached,
        # and 70B-shaped heads with 20 chunks of which about 14 are cached.
        dict(name="topk10-attn", op="attn", heads="llama8b", batch=8, prefix=3136, suffix=2112),
        dict(name="llama70b-long-attn", op="attn", heads="llama70b", batch=8, prefix=7232, suffix=3136),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        op = rng.choice(["qkv", "append", "attn", "split", "fused", "layer", "step"])
        if op == "step" or (op in ("qkv", "append", "attn", "fused") and rng.random() < 0.2):
            case = dict(op=op, heads="llama8b", trace=True, batch=log_int(1, 16), trace_seed=rng.randrange(1, 1000),
                        chunk=rng.choice([64, 128, 200, 256, 333]))
        else:
            case = dict(op=op, heads=rng.choice(sorted(HEADS)), batch=log_int(1, 24), suffix=log_int(1, 3000),
                        prefix=0 if rng.random() < 0.15 else BS * log_int(1, 450), spread=True,
                        shape_seed=rng.randrange(1000))
            if op in ("qkv", "layer"):
                case["bias"] = rng.random() < 0.5
            # short suffixes of few requests are what the split call is for
            if op == "split" and case["batch"] * case["suffix"] > 2000:
                continue
        s = work(case)
        if s["flops"] <= 2e12 and s["bytes"] <= 1.5e9:
            return case


class _Shape:
    """Host description of a case's batch."""

    def __init__(self, case, seed):
        self.hq, self.hkv, self.D, self.hidden = HEADS[case["heads"]]
        self.scale = self.D ** -0.5
        self.snapshot = self.prompts = None
        if case.get("trace"):
            # 64 queries were served before the batch; the pool's prefix matches
            # of the batch give its lengths
            self.w = w = W.llama8b_trace_batch(case.get("trace_seed", 0), case["batch"],
                                               chunk_tokens=case.get("chunk", 256))
            w.free_order_key = (int(seed),)   # physical placement
            self.stride = B.bt_stride_for(w)
            self.num_blocks = w.num_blocks()
            self.snapshot = cw.Pool(self.num_blocks, w.free_order())
            for p in w.warmup:
                got = cw.schedule_batch(self.snapshot, [p.tokens(0)], self.stride)
                cw.release_batch(self.snapshot, *got)
            self.prompts = [p.tokens(0) for p in w.prompts]
            pool = self.snapshot.clone()
            self.bt, self.plen, self.cu = cw.schedule_batch(pool, self.prompts, self.stride)
            return
        r = random.Random(case.get("shape_seed", 0))
        n = case["batch"]
        if case.get("spread"):
            S = [max(1, round(case["suffix"] * r.uniform(0.5, 1.5))) for _ in range(n)]
            P = [BS * round(case["prefix"] * r.uniform(0.5, 1.5) / BS) for _ in range(n)]
        else:
            S, P = [case["suffix"]] * n, [case["prefix"]] * n
        self.cu = np.concatenate([[0], np.cumsum(S)]).astype(np.int32)
        self.plen = np.asarray(P, np.int32)
        nblk = [-(-(p + s) // BS) for p, s in zip(P, S)]
        self.stride = max(nblk)
        self.num_blocks = sum(nblk) + 8
        order = np.random.default_rng(int(seed)).permutation(self.num_blocks).astype(np.int32)
        self.bt = np.full((n, self.stride), -1, np.int32)
        o = 0
        for i, k in enumerate(nblk):
            self.bt[i, :k] = order[o:o + k]
            o += k

    @property
    def rows(self):
        return int(self.cu[-1])

    def blocks(self, r):
        """Physical blocks of request r's prompt."""
        n = int(self.plen[r]) + int(self.cu[r + 1] - self.cu[r])
        return self.bt[r, :-(-n // BS)]


def _inputs(case, seed):
    """Shape and device tensors of a case, a function of the seed alone."""
    s = _Shape(case, seed)
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 7919 + 17)

    def normal(*shape, std=1.0):
        return (torch.randn(shape, generator=g, device="cuda") * std).to(torch.bfloat16)

    t = {"k_cache": normal(s.num_blocks, s.hkv, BS, s.D), "v_cache": normal(s.num_blocks, s.hkv, BS, s.D)}
    if case["op"] in ("qkv", "layer"):
        feats = (s.hq + 2 * s.hkv) * s.D
        t["x"] = normal(s.rows, s.hidden)
        t["w"] = normal(feats, s.hidden, std=s.hidden ** -0.5)
        t["bias"] = normal(feats, std=0.5) if case.get("bias") else None
    else:
        t["q"] = normal(s.rows, s.hq, s.D)
    if case["op"] in ("append", "fused", "step"):
        t["k_new"], t["v_new"] = normal(s.rows, s.hkv, s.D), normal(s.rows, s.hkv, s.D)
    return s, t


def _uses_split(meta):
    return cw.split_count(meta) > 1


def prepare(case, seed):
    s, t = _inputs(case, seed)
    op = case["op"]
    st = dict(t, op=op, shape=s)
    if op != "append":
        st["out"] = torch.empty((s.rows, s.hq, s.D), dtype=torch.bfloat16, device="cuda")
    if op == "step":
        rn = cw.BatchRunner(s.prompts, s.stride, s.hq, s.hkv, s.D, fused=True)
        rn.bind(t["q"], t["k_new"], t["v_new"], t["k_cache"], t["v_cache"], st["out"], s.scale)
        st.update(runner=rn, copies=torch.cuda.Stream(), up=None, done=None)
        return st
    st["meta"] = meta = cw.BatchMeta(s.bt, s.cu, s.plen, s.hq, s.hkv, s.D)
    if op in ("qkv", "layer"):
        last = int((s.plen + np.diff(s.cu)).max())
        st["rope"] = torch.from_numpy(cw.rope_table(last, s.D, ROPE_BASE)).cuda()
        st["q"] = torch.empty((s.rows, s.hq, s.D), dtype=torch.bfloat16, device="cuda")
    if op == "split" or (op == "layer" and _uses_split(meta)):
        n = cw.split_count(meta)
        meta.split_plan(n)
        st["workspace"] = torch.empty(max(1, cw.split_workspace_bytes(meta, n)), dtype=torch.uint8, device="cuda")
    if op == "fused":
        meta.append_plan(s.num_blocks)
    return st


def run(st):
    op, s = st["op"], st["shape"]
    kc, vc = st["k_cache"], st["v_cache"]
    if op == "step":
        return _run_step(st)
    meta = st["meta"]
    if op in ("qkv", "layer"):
        cw.qkv_rope_append(meta, st["x"], st["w"], st["rope"], kc, vc, bias=st["bias"], q_out=st["q"])
        if op == "qkv":
            return {"q": st["q"], "k_cache": kc, "v_cache": vc}
    if op == "append":
        cw.kv_append(meta, st["k_new"], st["v_new"], kc, vc)
        return {"k_cache": kc, "v_cache": vc}
    if op == "fused":
        cw.suffix_prefill_append_attn(meta, st["q"], st["k_new"], st["v_new"], kc, vc, s.scale, out=st["out"])
        return {"out": st["out"], "k_cache": kc, "v_cache": vc}
    if "workspace" in st:
        cw.suffix_prefill_attn_split(meta, st["q"], kc, vc, s.scale, workspace=st["workspace"], out=st["out"])
    else:
        cw.suffix_prefill_attn(meta, st["q"], kc, vc, s.scale, out=st["out"])
    if op == "layer":
        return {"out": st["out"], "q": st["q"], "k_cache": kc, "v_cache": vc}
    return {"out": st["out"]}


def _run_step(st):
    """One step of a serving loop: the schedule goes up on a copy stream; the
    pinned buffer is rewritten only once its last upload is done."""
    rn, copies, main = st["runner"], st["copies"], torch.cuda.current_stream()
    if st["up"] is not None:
        st["up"].synchronize()
    pool = st["shape"].snapshot.clone()
    rn.schedule(pool)
    with torch.cuda.stream(copies):
        if st["done"] is not None:
            copies.wait_event(st["done"])
        rn.upload()
        st["up"] = torch.cuda.Event()
        st["up"].record(copies)
    main.wait_event(st["up"])
    rn.append_attention()
    st["done"] = torch.cuda.Event()
    st["done"].record(main)
    rn.release(pool)
    pool.close()
    return {"out": st["out"], "k_cache": st["k_cache"], "v_cache": st["v_cache"]}


def work(case):
    s = _Shape(case, 0)
    op = case["op"]
    S, P = np.diff(s.cu).astype(np.int64), s.plen.astype(np.int64)
    T = int(S.sum())
    row_kv, row_q = s.hkv * s.D * 2, s.hq * s.D * 2
    feats = (s.hq + 2 * s.hkv) * s.D
    qkv = {"bytes": T * s.hidden * 2 + feats * s.hidden * 2 + T * (row_q + 2 * row_kv),
           "flops": 2 * T * s.hidden * feats}
    if op == "qkv":
        return qkv
    if op == "append":
        return {"bytes": 4 * T * row_kv, "flops": 0}
    # keys and values once per distinct physical block
    kv_rows = BS * len(np.unique(np.concatenate([s.blocks(r) for r in range(len(P))])))
    attn = {"bytes": 2 * T * row_q + 2 * kv_rows * row_kv,
            "flops": 4 * s.D * s.hq * int((S * P + S * (S + 1) // 2).sum())}
    if op in ("fused", "step"):
        attn["bytes"] += 2 * T * row_kv
    if op == "layer":
        attn = {k: attn[k] + qkv[k] for k in attn}
    return attn


def tolerance(case):
    op = case["op"]
    if op == "append":
        return "exact"   # a bit copy
    if op == "qkv":
        return {"rel": 4e-3, "max": 0.016}   # one bf16 rounding of a 32-bit sum
    # bf16 queries (scaled), probabilities and output around 32-bit sums
    return {"rel": 1e-2, "max": 0.1}


def exact(case, seed):
    s, t = _inputs(case, seed)
    op = case["op"]
    pos = np.concatenate([np.arange(p, p + n) for p, n in zip(s.plen, np.diff(s.cu))])
    req = np.repeat(np.arange(len(s.plen)), np.diff(s.cu))
    dev = "cuda"
    blk = torch.from_numpy(s.bt[req, pos // BS].astype(np.int64)).to(dev)
    slot = torch.from_numpy((pos % BS).astype(np.int64)).to(dev)

    def image(cache, rows):
        """The cache with the suffix rows [T, Hkv, D] in their slots."""
        c = cache.to(rows.dtype)
        c[blk, :, slot] = rows
        return c

    if op in ("qkv", "layer"):
        y = t["x"].double() @ t["w"].double().t()
        if t["bias"] is not None:
            y += t["bias"].double()
        y = y.view(s.rows, s.hq + 2 * s.hkv, s.D)
        half = s.D // 2
        theta = ROPE_BASE ** (-2.0 * torch.arange(half, dtype=torch.float64, device=dev) / s.D)
        ang = (torch.from_numpy(pos.astype(np.float64)).to(dev)[:, None] * theta)[:, None, :]
        c, sn = ang.cos(), ang.sin()
        rot = y[:, :s.hq + s.hkv]
        rot = torch.cat([rot[..., :half] * c - rot[..., half:] * sn, rot[..., half:] * c + rot[..., :half] * sn], -1)
        q, k, v = rot[:, :s.hq], rot[:, s.hq:], y[:, s.hq + s.hkv:]
        res = {"q": q.contiguous(), "k_cache": image(t["k_cache"], k), "v_cache": image(t["v_cache"], v)}
        if op == "qkv":
            return res
        # attention reads the stored (bfloat16) queries, keys and values
        q, kc, vc = (res[n].to(torch.bfloat16) for n in ("q", "k_cache", "v_cache"))
        res["out"] = _attention(s, q, kc, vc)
        return res
    kc, vc = t["k_cache"], t["v_cache"]
    if op in ("append", "fused", "step"):
        kc, vc = image(kc, t["k_new"]), image(vc, t["v_new"])
    if op == "append":
        return {"k_cache": kc, "v_cache": vc}
    out = _attention(s, t["q"], kc, vc)
    if op in ("fused", "step"):
        return {"out": out, "k_cache": kc, "v_cache": vc}
    return {"out": out}


def _attention(s, q, k_cache, v_cache):
    """Causal attention of the suffix rows over prefix and suffix, in float64."""
    out = torch.empty(q.shape, dtype=torch.float64, device=q.device)
    G = s.hq // s.hkv
    for r in range(len(s.plen)):
        c0, c1, P = int(s.cu[r]), int(s.cu[r + 1]), int(s.plen[r])
        L = P + c1 - c0
        ids = torch.from_numpy(s.blocks(r).astype(np.int64)).to(q.device)
        keys = torch.arange(L, device=q.device)
        for g in range(s.hkv):
            k = k_cache[ids, g].reshape(-1, s.D)[:L].double()
            v = v_cache[ids, g].reshape(-1, s.D)[:L].double()
            step = max(1, (1 << 26) // (G * L))
            for a in range(c0, c1, step):
                b = min(c1, a + step)
                sc = q[a:b, g * G:(g + 1) * G].double().reshape(-1, s.D) @ k.t() * s.scale
                sc = sc.view(b - a, G, L)
                hidden = keys[None, :] > P + torch.arange(a - c0, b - c0, device=q.device)[:, None]
                sc.masked_fill_(hidden[:, None, :], -math.inf)
                out[a:b, g * G:(g + 1) * G] = (torch.softmax(sc, -1).view(-1, L) @ v).view(b - a, G, s.D)
    return out
