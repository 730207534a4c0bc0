"""The work a decode lane has this library do, as cases that can be timed and checked.

A case is a dict of plain values; `listed()` gives the fixed ones, `draw(rng)` more of the same ranges.
`prepare(case, seed)` puts a batch on the GPU the way a serving program holds it (paged cache, block table,
queries, logits, outputs, workspaces), `run(state)` makes one pass through the public calls of
`paper_2604_09562_amd.binding`, `exact(case, seed)` gives the same results in 64 bits in plain torch.

Kinds: "attn" one verify-attention call, "accept" one acceptance call (chain or tree drafts), "step" a whole
decode step (append, attention per layer, acceptance, compaction for trees, commit).

Request lengths and depths follow from the case alone (its "sizes" number); the seed shuffles the requests and
makes every value.  Lengths and depths are spread as in the synthetic workloads of the package: uniform, or
uniform in the logarithm, never rounded to whole cache blocks.
"""
from __future__ import annotations

import math
import random

import torch

from paper_2604_09562_amd import binding

DEV = "cuda:0"
BLOCK = 16          # tokens per cache block
OUT_WIDTH = 21      # out_tokens row width
MAX_DEPTH = 20

_ESZ = {"f32": 4, "bf16": 2, "fp8": 1}


# ---------------------------------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------------------------------
def _attn(name, batch, ctx, lo, hi, k_lo, k_hi, hq, hkv, d, kv, q="bf16", tree=False, sizes=1):
    c = dict(kind="attn", batch=batch, ctx=ctx, ctx_lo=lo, ctx_hi=hi, depth_lo=k_lo, depth_hi=k_hi, hq=hq, hkv=hkv,
             head_dim=d, kv=kv, q=q, tree=tree, sizes=sizes)
    return dict(name=name, **c) if name else c


def _accept(name, batch, k_lo, k_hi, vocab, mode, logits="bf16", temperature=1.0, sigma_lo=1.0, sigma_hi=1.0, spike=0.0,
            ratio=False, sizes=1):
    c = dict(kind="accept", batch=batch, depth_lo=k_lo, depth_hi=k_hi, vocab=vocab, mode=mode, logits=logits,
             temperature=temperature, sigma_lo=sigma_lo, sigma_hi=sigma_hi, spike=spike, ratio=ratio, sizes=sizes)
    return dict(name=name, **c) if name else c


def _step(name, batch, ctx, lo, hi, k_lo, k_hi, hq, hkv, kv, layers, vocab, mode, temperature=0.8, sizes=1):
    c = dict(kind="step", batch=batch, ctx=ctx, ctx_lo=lo, ctx_hi=hi, depth_lo=k_lo, depth_hi=k_hi, hq=hq, hkv=hkv,
             head_dim=128, kv=kv, q="bf16", tree=mode.startswith("tree"), layers=layers, vocab=vocab, mode=mode, logits="bf16",
             temperature=temperature, sigma_lo=1.0, sigma_hi=1.0, spike=8.0, ratio=False, sizes=sizes)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # a nearly idle lane: four short requests; launches and latency decide
        _attn("attn_small_b4", 4, "uniform", 40, 600, 0, 8, 32, 8, 128, "bf16"),
        # the ordinary micro-batch of the benchmark: 64 requests at a fixed depth
        _attn("attn_8b_b64", 64, "uniform", 256, 4096, 4, 4, 32, 8, 128, "bf16"),
        # mixed traffic: many short and a few long requests, depths set per request by the controller
        _attn("attn_ragged_b128", 128, "log", 128, 16384, 0, 8, 32, 8, 128, "bf16"),
        # long documents: few requests, the cache is all that counts
        _attn("attn_long_b16", 16, "uniform", 16384, 65536, 6, 6, 32, 8, 128, "bf16"),
        # a large model with an 8-bit cache and eight query heads per KV head
        _attn("attn_70b_fp8_b96", 96, "uniform", 512, 8192, 2, 8, 64, 8, 128, "fp8"),
        # draft trees of 8 to 16 nodes
        _attn("attn_tree_b32", 32, "uniform", 256, 4096, 8, 16, 32, 8, 128, "bf16", tree=True),
        # the small float32 configuration with 64-wide heads
        _attn("attn_f32_b4", 4, "log", 64, 512, 4, 4, 8, 2, 64, "f32", q="f32"),
        # sampled acceptance on the ordinary micro-batch, with the ratios reported
        _accept("accept_8b_b64", 64, 4, 4, 128256, "sample", temperature=0.8, spike=8.0, ratio=True),
        # greedy acceptance of mixed traffic
        _accept("accept_greedy_b128", 128, 0, 8, 128256, "greedy", sigma_lo=0.3, sigma_hi=3.0),
        # sampled acceptance over draft trees
        _accept("accept_tree_b64", 64, 4, 4, 128256, "tree_sample", temperature=0.8, spike=8.0, ratio=True),
        # a whole decode step of a small lane: 8 requests, four layers, small vocabulary
        _step("step_b8_l4", 8, "uniform", 200, 1500, 2, 6, 32, 8, "bf16", 4, 32000, "sample"),
        # a whole decode step with draft trees and an 8-bit cache: greedy walk and compaction
        _step("step_tree_fp8_b16_l2", 16, "uniform", 512, 8192, 4, 8, 64, 8, "fp8", 2, 152064, "tree_greedy"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges: any batch size, grouping, cache type, depth, vocabulary; bounded in cost."""
    while True:
        kind = rng.choice(["attn"] * 5 + ["vector", "accept", "accept", "accept", "tree", "step", "step"])
        sizes = rng.randrange(1, 1 << 20)
        k_hi = rng.choice([0, 2, 3, 4, 5, 6, 7, 8, 8, 10, 12, 16, 20])
        k_lo = rng.randint(0, k_hi)
        hi = _log_int(rng, 64, 65536)
        lo = max(1, _log_int(rng, max(1, hi // 64), hi))
        if kind == "attn":
            kv = rng.choice(["bf16", "bf16", "fp8"])
            hkv = rng.choice([1, 2, 4, 8, 8])
            c = _attn(None, _log_int(rng, 1, 160), rng.choice(["uniform", "log"]), lo, hi, k_lo, k_hi,
                      hkv * rng.choice([1, 2, 4, 4, 8, 8]), hkv, 128, kv, tree=rng.random() < 0.25 and k_hi > 0, sizes=sizes)
            rows = (k_hi + 1) * c["hq"] // hkv
            if work(c)["bytes"] * (1 if rows <= 80 else 3) * (2 if kv == "fp8" else 1) > 2.0e9:
                continue
        elif kind == "vector":   # float32 or 64-wide heads or other groupings: small calls only
            hkv = rng.choice([1, 2, 4])
            d = rng.choice([64, 128])
            kv = rng.choice(["f32", "f32", "bf16", "fp8"])
            groups = [1, 2, 4, 7, 8] if d == 64 or kv == "f32" else [3, 5, 6, 7]
            c = _attn(None, _log_int(rng, 1, 8), "log", max(1, min(lo, 512) // 4), min(hi, 512), min(k_lo, 4), min(k_hi, 8),
                      hkv * rng.choice(groups), hkv, d, kv, q="f32" if kv == "f32" else "bf16", sizes=sizes)
        elif kind == "accept":
            c = _accept(None, _log_int(rng, 1, 128), k_lo, k_hi, _log_int(rng, 1000, 152064),
                        rng.choice(["sample", "sample", "greedy", "tree_greedy"]), logits=rng.choice(["bf16", "bf16", "f32"]),
                        temperature=rng.choice([0.7, 0.8, 1.0]), sigma_lo=0.3, sigma_hi=rng.choice([0.8, 3.0]),
                        spike=rng.choice([0.0, 8.0]), ratio=rng.random() < 0.5, sizes=sizes)
            if work(c)["bytes"] > 3.2e8:
                continue
        elif kind == "tree":
            c = _accept(None, _log_int(rng, 1, 64), k_lo, min(k_hi, 6), _log_int(rng, 1000, 152064), "tree_sample",
                        logits=rng.choice(["bf16", "bf16", "f32"]), temperature=rng.choice([0.7, 1.0]), sigma_lo=0.3, sigma_hi=1.5,
                        ratio=rng.random() < 0.5, sizes=sizes)
            c["depth_lo"] = min(c["depth_lo"], c["depth_hi"])
            if work(c)["bytes"] > 1.6e8:
                continue
        else:
            mode = rng.choice(["sample", "greedy", "tree_greedy"])
            hkv = rng.choice([4, 8])
            c = _step(None, _log_int(rng, 2, 24), "uniform", min(lo, 4096), min(hi, 4096), min(k_lo, 8), min(k_hi, 8),
                      hkv * rng.choice([4, 8]), hkv, rng.choice(["bf16", "fp8"]), rng.randint(1, 3), _log_int(rng, 8000, 152064), mode,
                      sizes=sizes)
            if work(c)["bytes"] > 6.0e8:
                continue
        return c


# ---------------------------------------------------------------------------------------------------
# sizes: from the case alone
# ---------------------------------------------------------------------------------------------------
def _sizes(case):
    """[(cache length counting the new tokens, draft depth)] per request, before shuffling."""
    rng = random.Random(case["sizes"])
    out = []
    for _ in range(case["batch"]):
        k = rng.randint(case["depth_lo"], case["depth_hi"])
        n = 0
        if case["kind"] != "accept":
            lo, hi = case["ctx_lo"], case["ctx_hi"]
            n = rng.randint(lo, hi) if case["ctx"] == "uniform" else _log_int(rng, lo, hi)
            n = max(n, k + 1)
        out.append((n, k))
    return out


def _shuffled(case, seed):
    s = _sizes(case)
    random.Random(seed * 7919 + 1).shuffle(s)
    return s


def _work_attn(case, sizes):
    hq, hkv, d, es = case["hq"], case["hkv"], case["head_dim"], _ESZ[case["kv"]]
    qs = 4 if case["q"] == "f32" else 2
    tokens = sum(n for n, _ in sizes)
    blocks = sum((n + BLOCK - 1) // BLOCK for n, _ in sizes)
    rows = sum(k + 1 for _, k in sizes)
    byts = tokens * hkv * d * 2 * es + blocks * 4 + rows * hq * (2 * d * qs + 4) + 8 * len(sizes)
    if case["kv"] == "fp8":
        byts += blocks * hkv * 8
    flops = sum(4 * d * hq * ((k + 1) * (n - k - 1) + (k + 1) * (k + 2) // 2) for n, k in sizes)
    return byts, flops


def _work_accept(case, sizes):
    rows = sum(k + 1 for _, k in sizes)
    if case["mode"] in ("sample", "tree_sample"):
        rows += sum(k for _, k in sizes)
    byts = rows * case["vocab"] * _ESZ[case["logits"]] + len(sizes) * 4 * (OUT_WIDTH + 1)
    return byts, 4 * rows * case["vocab"]


def work(case):
    sizes = _sizes(case)
    if case["kind"] == "attn":
        b, f = _work_attn(case, sizes)
    elif case["kind"] == "accept":
        b, f = _work_accept(case, sizes)
    else:
        b, f = _work_attn(case, sizes)
        new = sum(k + 1 for _, k in sizes) * case["hkv"] * case["head_dim"] * 2
        b = case["layers"] * (b + new * (2 + _ESZ[case["kv"]]))
        f *= case["layers"]
        b2, f2 = _work_accept(case, sizes)
        b, f = b + b2, f + f2
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------------------------------------------
# inputs: from case and seed
# ---------------------------------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _int32(values):
    return torch.tensor(values, dtype=torch.int32, device=DEV)


def _trees(sizes, seed):
    """A random draft tree per request: parent of node i drawn from 0..i-1; mask bit j = ancestor or self."""
    rng = random.Random(seed * 7919 + 2)
    parent, mask = [], []
    for _, k in sizes:
        own = [1]
        parent.append(-1)
        for i in range(1, k + 1):
            p = rng.randrange(i)
            parent.append(p)
            own.append(own[p] | (1 << i))
        mask += own
    return parent, mask


def _cache_values(shape, dtype, gen):
    """N(0,1) keys or values in storage format: (data, per-block scale or None)."""
    if dtype == "bf16":
        return torch.randn(shape, dtype=torch.bfloat16, device=DEV, generator=gen).view(torch.int16), None
    if dtype == "f32":
        return torch.randn(shape, dtype=torch.float32, device=DEV, generator=gen), None
    scale = torch.rand(shape[:2], device=DEV, generator=gen) * 0.09 + 0.01
    data = torch.empty(shape, dtype=torch.uint8, device=DEV)
    for lo in range(0, shape[0], 8192):
        s = scale[lo:lo + 8192, :, None, None]
        x = torch.randn((s.shape[0],) + tuple(shape[1:]), device=DEV, generator=gen) / s
        data[lo:lo + 8192] = x.clamp_(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8)
    return data, scale


def _attention_inputs(case, seed, sizes, gen, layer=0):
    """One layer's batch as the dict of device tensors and sizes that the attention calls take."""
    B, hq, hkv, d = case["batch"], case["hq"], case["hkv"], case["head_dim"]
    blocks = [(n + BLOCK - 1) // BLOCK for n, _ in sizes]
    used, most = sum(blocks), max(blocks)
    num_blocks = used + used // 10 + 1
    perm = torch.randperm(num_blocks, generator=torch.Generator().manual_seed(seed))[:used].to(torch.int32)
    table = torch.full((B, most), -1, dtype=torch.int32)
    at = 0
    for b, n in enumerate(blocks):
        table[b, :n] = perm[at:at + n]
        at += n
    indptr = [0]
    for _, k in sizes:
        indptr.append(indptr[-1] + k + 1)
    R = indptr[-1]
    shape = (num_blocks, hkv, BLOCK, d)
    k_cache, k_scale = _cache_values(shape, case["kv"], gen)
    v_cache, v_scale = _cache_values(shape, case["kv"], gen)
    # the slots behind a request's last token hold garbage, as in a cache in use
    big = {"f32": 1.0e4, "bf16": 0x461C, "fp8": 0x7E}[case["kv"]]
    for r in range(1, BLOCK):
        last = [int(table[b, blocks[b] - 1]) for b in range(B) if sizes[b][0] % BLOCK == r]
        if last:
            ids = torch.tensor(last, device=DEV)
            k_cache[ids, :, r:, :] = big
            v_cache[ids, :, r:, :] = big
    # heads differ in how sharply they attend
    sharp = torch.rand((1, hq, 1), device=DEV, generator=gen) * 3.0 + 1.0
    q = torch.randn((R, hq, d), device=DEV, generator=gen) * sharp
    q = q if case["q"] == "f32" else q.to(torch.bfloat16).view(torch.int16)
    inp = dict(batch=B, num_q_heads=hq, num_kv_heads=hkv, head_dim=d, block_size=BLOCK, num_blocks=num_blocks,
               max_blocks_per_seq=most, total_rows=R, kv_dtype=case["kv"], q_dtype=case["q"], kv_len=_int32([n for n, _ in sizes]),
               q_indptr=_int32(indptr), block_table=table.to(DEV), k_cache=k_cache, v_cache=v_cache, k_scale=k_scale,
               v_scale=v_scale, q=q, sm_scale=1.0 / math.sqrt(d))
    if case["tree"]:
        inp["tree_mask"] = _int32(_trees(sizes, seed)[1])
    return inp


def _accept_inputs(case, seed, sizes, gen):
    """Target and draft logits, draft tokens and uniforms, as the model, the draft model and the sampler leave them."""
    B, V, mode = case["batch"], case["vocab"], case["mode"]
    stride = (V + 7) // 8 * 8
    k = [x for _, x in sizes]
    indptr = [0]
    for x in k:
        indptr.append(indptr[-1] + x + 1)
    R, Rd = indptr[-1], indptr[-1] - B
    dt = torch.bfloat16 if case["logits"] == "bf16" else torch.float32
    target = torch.randn((R, stride), device=DEV, generator=gen) * 3.0
    if case["spike"]:
        hot = torch.randint(0, V, (R, 1), device=DEV, generator=gen)
        target.scatter_add_(1, hot, torch.full((R, 1), case["spike"], device=DEV))
    target = target.to(dt)
    tree = mode.startswith("tree")
    parent = _trees(sizes, seed)[0] if tree else None
    # the target row each draft is judged by: the row before it in a chain, its parent's row in a tree
    judge = [indptr[b] + (parent[indptr[b] + i + 1] if tree else i) for b in range(B) for i in range(k[b])]
    sigma = torch.rand((B,), device=DEV, generator=gen) * (case["sigma_hi"] - case["sigma_lo"]) + case["sigma_lo"]
    draft = torch.empty((max(Rd, 1), stride), dtype=dt, device=DEV)
    tokens = torch.zeros((max(Rd, 1),), dtype=torch.int32, device=DEV)
    if Rd:
        jt = torch.tensor(judge, device=DEV)
        src = sorted(set(judge)) if tree else judge            # siblings in a tree come from one proposal
        where = {j: i for i, j in enumerate(src)}
        pick = torch.tensor([where[j] if tree else i for i, j in enumerate(judge)], device=DEV)
        owner = torch.tensor([b for b in range(B) for _ in range(k[b])], device=DEV)
        noise = torch.randn((len(src), stride), device=DEV, generator=gen)
        for lo in range(0, Rd, 256):
            s = slice(lo, min(lo + 256, Rd))
            x = (target[jt[s]].float() + noise[pick[s]] * sigma[owner[s], None]).to(dt)
            draft[s] = x
            if mode in ("sample", "tree_sample"):
                p = torch.softmax(x[:, :V].float() / case["temperature"], dim=1)
                tokens[s] = torch.multinomial(p, 1, generator=gen)[:, 0].to(torch.int32)
            elif mode == "greedy":
                tokens[s] = x[:, :V].float().argmax(dim=1).to(torch.int32)
            else:   # a candidate is often what greedy decoding emits after its parent
                best = target[jt[s]][:, :V].float().argmax(dim=1)
                other = torch.randint(0, V, best.shape, device=DEV, generator=gen)
                hit = torch.rand(best.shape, device=DEV, generator=gen) < 0.6
                tokens[s] = torch.where(hit, best, other).to(torch.int32)
        del noise
    greedy = mode in ("greedy", "tree_greedy")
    inp = dict(batch=B, vocab=V, row_stride=stride, logit_dtype=case["logits"], total_rows=R, q_indptr=_int32(indptr),
               target_logits=target, draft_logits=draft, draft_tokens=tokens,
               u_accept=torch.rand((max(Rd, 1),), device=DEV, generator=gen), u_sample=torch.rand((B,), device=DEV, generator=gen),
               temperature=torch.full((B,), case["temperature"], device=DEV), greedy=int(greedy))
    if tree:
        inp["tree_parent"] = _int32(parent)
    return inp


def _inputs(case, seed):
    sizes = _shuffled(case, seed)
    gen = _gen(seed)
    got = {"sizes": sizes}
    if case["kind"] == "attn":
        got["layers"] = [_attention_inputs(case, seed, sizes, gen)]
    elif case["kind"] == "step":
        got["layers"] = [_attention_inputs(case, seed, sizes, gen) for _ in range(case["layers"])]
        first = got["layers"][0]
        for d in got["layers"]:   # the layers of a step share block table, lengths and offsets
            for name in ("block_table", "kv_len", "q_indptr", "tree_mask"):
                if name in first:
                    d[name] = first[name]
            shape = (d["total_rows"], case["hkv"], case["head_dim"])
            d["new_dtype"] = "bf16"
            d["k_new"] = torch.randn(shape, dtype=torch.bfloat16, device=DEV, generator=gen)
            d["v_new"] = torch.randn(shape, dtype=torch.bfloat16, device=DEV, generator=gen)
    if case["kind"] != "attn":
        got["accept"] = _accept_inputs(case, seed, sizes, gen)
    return got


def prepare(case, seed):
    st = _inputs(case, seed)
    st["case"] = case
    st["max_q_len"] = max(k for _, k in st.pop("sizes")) + 1   # the bound a caller has from its depth controller
    mq = st["max_q_len"]
    if "layers" in st:
        st["out"], st["lse"] = [], []
        for d in st["layers"]:
            out, lse, ws = binding.alloc_attention_outputs(d, DEV, max_q_len=mq)
            st["out"].append(out)
            st["lse"].append(lse)
            st.setdefault("ws_attn", ws)   # one workspace serves the layers of a step, which share their plan
    if "accept" in st:
        d = st["accept"]
        st["accepted"], st["tokens"], ratio, st["ws_accept"] = binding.alloc_accept_outputs(d, DEV)
        st["ratio"] = ratio if case["ratio"] and case["mode"] in ("sample", "tree_sample") else None
        if case["mode"].startswith("tree"):
            st["nodes"] = torch.empty((d["batch"], MAX_DEPTH), dtype=torch.int32, device=DEV)
        if case["mode"] == "tree_sample":
            st["ws_accept"] = binding.tree_sample_workspace(d, DEV)
    if case["kind"] == "step":
        st["kv_len_next"] = torch.empty_like(st["layers"][0]["kv_len"])
    return st


# ---------------------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------------------
def _values(out, case):
    return out if case["q"] == "f32" else out.view(torch.bfloat16)


def _run_accept(st):
    d, mq, mode = st["accept"], st["max_q_len"], st["case"]["mode"]
    got = {"accepted": st["accepted"], "tokens": st["tokens"]}
    if mode == "tree_sample":
        binding.ss_spec_accept_tree_sample(d, st["accepted"], st["tokens"], st["nodes"], st["ratio"], st["ws_accept"], max_q_len=mq)
    elif mode == "tree_greedy":
        binding.ss_spec_accept_tree_greedy(d, st["accepted"], st["tokens"], st["nodes"], st["ws_accept"], max_q_len=mq)
    else:
        binding.ss_spec_accept(d, st["accepted"], st["tokens"], st["ratio"], st["ws_accept"], max_q_len=mq)
    if mode.startswith("tree"):
        got["nodes"] = st["nodes"]
    if st["ratio"] is not None:
        got["ratio"] = st["ratio"]
    return got


def run(st):
    case, mq = st["case"], st["max_q_len"]
    if case["kind"] == "attn":
        binding.ss_spec_verify_attn(st["layers"][0], st["out"][0], st["lse"][0], st["ws_attn"], max_q_len=mq)
        return {"out": _values(st["out"][0], case), "lse": st["lse"][0]}
    if case["kind"] == "accept":
        return _run_accept(st)
    for i, d in enumerate(st["layers"]):
        binding.ss_kv_append(d, max_q_len=mq)
        binding.ss_spec_verify_attn(d, st["out"][i], st["lse"][i], st["ws_attn"], max_q_len=mq, reuse_plan=i > 0)
    got = _run_accept(st)
    if "nodes" in got:
        for d in st["layers"]:
            binding.ss_kv_compact(d, st["nodes"], st["accepted"], max_q_len=mq)
    # the valid lengths after the step, in a buffer of their own: the next pass starts from the same ones
    st["kv_len_next"].copy_(st["layers"][0]["kv_len"])
    binding.ss_kv_commit(st["layers"][0]["q_indptr"], st["accepted"], st["kv_len_next"])
    got["kv_len"] = st["kv_len_next"]
    for i, d in enumerate(st["layers"]):
        got["out%d" % i] = _values(st["out"][i], case)
        got["lse%d" % i] = st["lse"][i]
        for name in ("k_cache", "v_cache", "k_scale", "v_scale"):
            if d[name] is not None:
                got["%s%d" % (name, i)] = d[name]
    return got


# Measured against exact(): bf16 attention is 1.9e-3 to 2.5e-3 off, output and probabilities being rounded to bf16;
# float32 attention is 6.4e-7 off, the ratios 3.3e-7 (sums in 32 bits).  About four times that is stated.  "differ"
# allows for a uniform that falls on a ratio or a boundary of the distribution within the rounding of 32-bit sums.
def tolerance(case):
    if case["kind"] == "accept":
        if case["mode"] in ("greedy", "tree_greedy"):
            return "exact"
        return {"rel": 2e-6, "max": 2e-5, "differ": 0.002}
    if case["q"] == "f32":
        return {"rel": 3e-6, "max": 3e-5}
    return {"rel": 1e-2, "max": 1e-1, "differ": 0.002 if case["kind"] == "step" else 0.0}


# ---------------------------------------------------------------------------------------------------
# the same results in 64 bits
# ---------------------------------------------------------------------------------------------------
def _decode(x, dtype):
    if dtype == "f32":
        return x.double()
    if dtype == "bf16":
        return x.view(torch.bfloat16).double()
    return x.view(torch.float8_e4m3fn).double()


def _store_new(case, d, sizes):
    """The append of a step, on the inputs' own cache tensors."""
    at = 0
    for b, (n, k) in enumerate(sizes):
        for side in ("k", "v"):
            cache, new = d[side + "_cache"], d[side + "_new"]
            pos = torch.arange(n - k - 1, n, device=DEV)
            phys = d["block_table"][b].long()[pos // BLOCK]
            rows = new[at:at + k + 1].float()
            if case["kv"] == "bf16":
                cache[phys, :, pos % BLOCK] = rows.to(torch.bfloat16).view(torch.int16)
                continue
            scale = d[side + "_scale"]
            for blk in sorted(set((pos // BLOCK).tolist())):
                inside = pos // BLOCK == blk
                p = int(d["block_table"][b, blk])
                if blk * BLOCK >= n - k - 1:   # the block begins with this step: its scale is set by the new tokens
                    amax = rows[inside].abs().amax(dim=(0, 2))
                    scale[p] = torch.where(amax > 0, amax / 448.0, torch.ones_like(amax))
                x = (rows[inside] / scale[p][None, :, None]).clamp(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8)
                cache[p, :, pos[inside] % BLOCK] = x.transpose(0, 1)
        at += k + 1


def _exact_attention(case, d, sizes):
    hq, hkv, dim = case["hq"], case["hkv"], case["head_dim"]
    G = hq // hkv
    out = torch.empty((d["total_rows"], hq, dim), dtype=torch.float64, device=DEV)
    lse = torch.empty((d["total_rows"], hq), dtype=torch.float64, device=DEV)
    q = _decode(d["q"], case["q"])
    at = 0
    for b, (n, k) in enumerate(sizes):
        ids = d["block_table"][b, :(n + BLOCK - 1) // BLOCK].long()
        kv = []
        for side in ("k", "v"):
            x = _decode(d[side + "_cache"][ids], case["kv"])
            if d[side + "_scale"] is not None:
                x = x * d[side + "_scale"][ids].double()[:, :, None, None]
            kv.append(x.permute(1, 0, 2, 3).reshape(hkv, -1, dim)[:, :n])
        rows = k + 1
        see = torch.ones((rows, n), dtype=torch.bool, device=DEV)
        if d.get("tree_mask") is not None:
            bits = d["tree_mask"][at:at + rows].long() & 0xFFFFFFFF
            see[:, n - rows:] = ((bits[:, None] >> torch.arange(rows, device=DEV)[None, :]) & 1).bool()
        else:
            see[:, n - rows:] = torch.tril(torch.ones((rows, rows), dtype=torch.bool, device=DEV))
        for h in range(hkv):
            kt = kv[0][h].t().contiguous()
            qh = q[at:at + rows, h * G:(h + 1) * G].reshape(rows * G, dim).contiguous()
            s = (qh @ kt) * d["sm_scale"]
            s = s.masked_fill(~see.repeat_interleave(G, dim=0), -math.inf)
            z = torch.logsumexp(s, dim=1)
            o = torch.exp(s - z[:, None]) @ kv[1][h].contiguous()
            out[at:at + rows, h * G:(h + 1) * G] = o.reshape(rows, G, dim)
            lse[at:at + rows, h * G:(h + 1) * G] = z.reshape(rows, G)
        at += rows
    return out, lse


def _exact_ratios(case, d, sizes):
    """p/q of every draft of a chain, r/q of every offered node of a tree (NaN where none was offered)."""
    V, T = case["vocab"], case["temperature"]
    T = float(torch.tensor(T, dtype=torch.float32))
    Rd = d["total_rows"] - d["batch"]
    ratio = torch.full((max(Rd, 1),), math.nan, dtype=torch.float64, device=DEV)
    soft = lambda rows, i: torch.softmax(rows[i, :V].double() / T, dim=0)   # noqa: E731
    u = d["u_accept"].double().tolist()
    tok = d["draft_tokens"].tolist()
    parent = d["tree_parent"].tolist() if case["mode"].startswith("tree") else None
    t0 = 0
    for b, (_, k) in enumerate(sizes):
        d0 = t0 - b
        if parent is None:
            for i in range(k):
                x = tok[d0 + i]
                ratio[d0 + i] = soft(d["target_logits"], t0 + i)[x] / soft(d["draft_logits"], d0 + i)[x]
        else:
            cur, r = 0, soft(d["target_logits"], t0)
            for c in range(1, k + 1):
                if parent[t0 + c] != cur:
                    continue
                qc, x = soft(d["draft_logits"], d0 + c - 1), tok[d0 + c - 1]
                ratio[d0 + c - 1] = r[x] / qc[x]
                if u[d0 + c - 1] * float(qc[x]) < float(r[x]):
                    cur, r = c, soft(d["target_logits"], t0 + c)
                else:
                    rest = (r - qc).clamp_(min=0.0)
                    if float(rest.sum()) > 0:
                        r = rest / rest.sum()
        t0 += k + 1
    return ratio


def exact(case, seed):
    """What run() returns, in 64 bits; None for whole values (tokens, lengths, cache bytes) and what depends on them."""
    st = _inputs(case, seed)
    sizes = st["sizes"]
    got = {}
    ratio = case["kind"] != "attn" and case["ratio"] and case["mode"] in ("sample", "tree_sample")
    if case["kind"] == "accept" and not ratio:
        return None
    if case["kind"] != "attn":
        got.update(accepted=None, tokens=None)
        if case["mode"].startswith("tree"):
            got["nodes"] = None
        if ratio:
            got["ratio"] = _exact_ratios(case, st["accept"], sizes)
    if case["kind"] == "attn":
        got["out"], got["lse"] = _exact_attention(case, st["layers"][0], sizes)
    if case["kind"] == "step":
        got["kv_len"] = None
        for i, d in enumerate(st["layers"]):
            _store_new(case, d, sizes)
            got["out%d" % i], got["lse%d" % i] = _exact_attention(case, d, sizes)
            for name in ("k_cache", "v_cache", "k_scale", "v_scale"):
                if d[name] is not None:
                    got["%s%d" % (name, i)] = None
    return got
