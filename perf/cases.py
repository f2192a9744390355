"""Timing cases of the tiered decode attention path, through the calls a decoding program makes:

  step     one decode step of one attention layer: append the new token, attend over every tier, check for eviction
  topk     the same with block identification: only the k best-scoring blocks of the last tier are attended
  prefill  a prompt tiered in one go: every tier's share quantized through the formats of the tiers above it
  evict    one eviction cascade: the oldest block of every full tier moves down, re-quantized

A case names the cache ("tiers": one entry per tier, newest first, K format / V format : tokens held : block tokens), the
batch, the head counts, the queries' type, where the last tier lives, whether its tiers are paged, and how ragged the
batch is.  Keys are N(0, 1) with every 50th (head, channel) pair scaled by 8, as the keys of trained models show;
values and queries N(0, 1)."""
import math
import random

import numpy as np
import torch

from paper_2604_19769_amd.cache import TierConfig, TieredCache

DEV = "cuda:0"
DT = {"f16": torch.float16, "bf16": torch.bfloat16}
BYTES = {"f16": 256, "bf16": 256, "i8": 136, "i4": 72, "i4c": 72, "i4t": 68}     # stored bytes per token of one KV head


def listed():
    def case(name, kind, batch, heads, tiers, q="f16", host=False, paged=False, ragged=1.0, select=0):
        hq, hkv = heads
        return {"name": name, "kind": kind, "batch": batch, "q_heads": hq, "kv_heads": hkv, "tiers": tiers, "q": q,
                "host": host, "paged": paged, "ragged": ragged, "select": select}

    return [
        # the smallest deployment: one short conversation on a small model; launches and host time are what it costs
        case("step_tiny_4k", "step", 1, (8, 2), "f16/f16:507:64 i8/i8:3584:64"),
        # multi-head model (7B shape), batch of four at 32K, compressed tier in HBM: the benchmark's main workload
        case("step_mha_32k", "step", 4, (32, 32), "f16/f16:1985:128 i4/i4:30720:128"),
        # one long document on an 8B grouped-query model, bf16, three tiers all in HBM: latency per token at 128K
        case("step_gqa_128k", "step", 1, (32, 8), "bf16/bf16:4001:128 i8/i8:28672:128 i4/i4:98304:1024", q="bf16"),
        # serving: sixteen conversations of unequal length, paged, values packed for the matrix cores
        case("step_serving_ragged", "step", 16, (32, 8), "f16/f16:4033:256 i8/i8:8192:256 i4/i4c:53248:256", paged=True, ragged=0.1),
        # serving at full batch with short contexts
        case("step_short_x64", "step", 64, (32, 8), "f16/f16:1003:128 i8/i8:3072:128", ragged=0.5),
        # the paper's own layout (fp16 window + K 8-bit / V 4-bit) on a model with sixteen query heads per KV head
        case("step_k8v4_wide", "step", 8, (64, 4), "f16/f16:2013:128 i8/i4:63488:128"),
        # the slow tier in pinned host memory, read over PCIe: the benchmark's offload workload
        case("step_offload_128k", "step", 1, (32, 8), "bf16/bf16:4001:128 i8/i8:28672:1024 i4/i4:98304:1024", q="bf16", host=True),
        # block-sparse recall at 128K: 64 of 96 blocks of the oldest tier
        case("topk_128k", "topk", 4, (32, 8), "f16/f16:4001:128 i8/i8:28672:1024 i4/i4:98304:1024", select=64),
        # prompts of a multi-head model tiered into fp16 + int4
        case("prefill_mha_8k", "prefill", 2, (32, 32), "f16/f16:2047:128 i4/i4:6144:128"),
        # prompts of a grouped-query model tiered three deep, mean keys kept for block identification
        case("prefill_gqa_summaries", "prefill", 4, (32, 8), "f16/f16:4095:128 i8/i8:8192:256 i4/i4:20480:256", select=1),
        # a prompt into the paper's formats with values packed for the matrix cores, bf16 model, paged
        case("prefill_k8v4c_bf16", "prefill", 1, (32, 8), "bf16/bf16:4095:128 i8/i4c:28672:256", q="bf16", paged=True),
        # what a decode loop of sixteen sequences pays when its tiers are full: one block of each moves down
        case("evict_x16", "evict", 16, (32, 8), "f16/f16:1024:128 i8/i8:2048:128 i4/i4:4096:256", select=1),
    ]


HEADS = ((8, 2), (32, 32), (16, 16), (32, 16), (24, 8), (32, 8), (48, 8), (64, 8), (28, 4), (64, 4), (64, 2))


def draw(rng: random.Random):
    while True:
        kind = rng.choices(("step", "topk", "prefill", "evict"), (6, 1, 3, 1))[0]
        hq, hkv = rng.choice(HEADS)
        batch = round(2 ** rng.uniform(0, 6))
        q = rng.choice(("f16", "f16", "bf16"))
        window = round(2 ** rng.uniform(8, 12)) + rng.randrange(64)
        old = round(2 ** rng.uniform(10, 17)) // 128 * 128
        quant = ["i8/i8", "i4/i4", "i8/i4"] + (["i8/i4c", "i4/i4c"] if hq > hkv else []) + ([] if hq > 4 * hkv else ["i4t/i4"])
        last = rng.choice(quant)
        if kind in ("topk", "evict"):
            last = rng.choice(("i8/i8", "i4/i4"))
        bt = rng.choice((128, 128, 256, 1024))
        tiers = ["%s/%s:%d:128" % (q, q, max(window, 256) // (128 if kind == "evict" else 1) * (128 if kind == "evict" else 1))]
        if rng.random() < 0.4 and last in ("i4/i4", "i4/i4c", "i4t/i4"):
            mid = max(1, round(old * rng.uniform(0.1, 0.4)) // 128) * 128
            tiers.append("i8/i8:%d:%d" % (mid, 128 if kind == "evict" else rng.choice((128, 256))))
            old = max(128, old - mid)
        tiers.append("%s:%d:%d" % (last, old, bt))
        case = {"kind": kind, "batch": batch, "q_heads": hq, "kv_heads": hkv, "tiers": " ".join(tiers), "q": q,
                "host": kind == "step" and rng.random() < 0.08, "paged": rng.random() < 0.3,
                "ragged": 1.0 if kind in ("evict", "prefill") else rng.choice((1.0, 0.6, 0.2)),
                "select": 0}
        if kind == "topk":
            blocks = (old + bt - 1) // bt
            if not 4 <= blocks <= 1024:
                continue
            case["select"] = max(1, round(blocks * rng.uniform(0.1, 0.7)))
        if kind in ("prefill", "evict"):
            case["select"] = int(last != "i4t/i4" and rng.random() < 0.4)
        w = work(case)["bytes"]
        if 1e6 <= w <= (1e8 if case["host"] else 5e8 if kind == "prefill" else 1e9) and held(case) <= 1.2e9:
            return case


# ------------------------------------------------------------------ shapes

def spec(case):
    """[(k_fmt, v_fmt, tokens, block_tokens)] per tier, newest first."""
    out = []
    for t in case["tiers"].split():
        f, n, bt = t.split(":")
        k, v = f.split("/")
        out.append((k, v, int(n), int(bt)))
    return out


def lengths(case):
    """Tokens held per tier and sequence: every tier but the last is as full as the case says, the last one ragged (in
    whole blocks of 128 tokens, as evictions deliver them)."""
    tiers, B = spec(case), case["batch"]
    out = [[n] * B for _, _, n, _ in tiers]
    if case["ragged"] < 1.0 and len(tiers) > 1:
        n = tiers[-1][2]
        for b in range(1, B):
            f = (b * 0.6180339887) % 1.0
            out[-1][b] = max(128, int(n * (case["ragged"] + (1.0 - case["ragged"]) * f)) // 128 * 128)
    return out


def held(case):
    """Bytes stored by the whole cache."""
    return case["kv_heads"] * sum(sum(ns) * (BYTES[k] + BYTES[v]) for ns, (k, v, _, _) in zip(lengths(case), spec(case)))


def evicted(case):
    """Blocks' tokens that leave each tier but the last in one cascade (per sequence)."""
    return [t[3] for t in spec(case)[:-1]]


def work(case):
    tiers, lens, B, hq, hkv = spec(case), lengths(case), case["batch"], case["q_heads"], case["kv_heads"]
    if case["kind"] == "prefill":
        n = sum(sum(x) for x in lens)
        return {"bytes": n * hkv * 512 + held(case), "flops": 0}
    if case["kind"] == "evict":
        moved = 0
        for t, n in enumerate(evicted(case)):
            moved += n * (BYTES[tiers[t][0]] + BYTES[tiers[t][1]] + BYTES[tiers[t + 1][0]] + BYTES[tiers[t + 1][1]])
        return {"bytes": B * hkv * moved, "flops": 0}
    tokens = [sum(x) for x in lens]
    extra = 0
    if case["kind"] == "topk":
        bt = tiers[-1][3]
        tokens[-1] = sum(min(n, min(case["select"], -(-n // bt)) * bt) for n in lens[-1])
        extra = sum(-(-n // bt) for n in lens[-1]) * hkv * 256                      # the mean keys
    kv = sum(n * (BYTES[k] + BYTES[v]) for n, (k, v, _, _) in zip(tokens, tiers)) * hkv
    return {"bytes": kv + extra + B * hq * (256 + 512 + 4) + B * hkv * 1024, "flops": 4 * 128 * sum(tokens) * (hq // hkv) * hkv}


def tolerance(case):
    if case["kind"] in ("prefill", "evict"):
        return "exact"
    # Measured against exact() and four times that: one query head per KV head (fp32 weights, exact codes) 6e-6, with
    # int4 codes 6.5e-5 (their scores are sums of some 1e4 whose offset leaves in fp32); grouped queries (softmax
    # weights and decompressed values rounded once to fp16) 2.3e-4.
    if case["q_heads"] != case["kv_heads"]:
        return {"rel": 1e-3, "max": 0.02}
    return {"rel": 2.6e-4, "max": 5e-3} if "i4" in case["tiers"] else {"rel": 2.5e-5, "max": 5e-4}


# ------------------------------------------------------------------ inputs

def generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1000003 + 17)
    return g


def normal(g, shape, dtype):
    return torch.randn(shape, generator=g, device=DEV, dtype=torch.float32).to(dtype)


def inputs(case, seed):
    """q, k_new, v_new, and per tier a list of (sequence or -1, K, V) to load, all from the seed."""
    B, hq, hkv, dt = case["batch"], case["q_heads"], case["kv_heads"], DT[case["q"]]
    g = generator(seed)
    scale = torch.ones(hkv * 128, device=DEV)
    scale[torch.randperm(hkv * 128, generator=g, device=DEV)[:max(1, hkv * 128 // 50)]] = 8.0
    scale = scale.view(hkv, 1, 128)

    def keys(*shape):
        return (torch.randn(shape, generator=g, device=DEV, dtype=torch.float32) * scale).to(dt)

    loads = []
    for lens in lengths(case):
        if len(set(lens)) == 1:
            loads.append([(-1, keys(B, hkv, lens[0], 128), normal(g, (B, hkv, lens[0], 128), dt))])
        else:
            loads.append([(b, keys(hkv, n, 128), normal(g, (hkv, n, 128), dt)) for b, n in enumerate(lens)])
    return normal(g, (B, hq, 128), dt), keys(B, hkv, 1, 128), normal(g, (B, hkv, 1, 128), dt), loads


def prepare(case, seed):
    tiers, B = spec(case), case["batch"]
    q, k_new, v_new, loads = inputs(case, seed)
    last = len(tiers) - 1
    cfg = []
    for t, (k, v, n, bt) in enumerate(tiers):
        evict = case["kind"] == "evict"
        # a window in steady state: evicting half a block from now, or (the eviction case) one block of every tier due
        cap = 10 ** 9 if t == last else max(bt, n + (tiers[t - 1][3] if t else 0) if evict else n + 64)
        ring = -(-(n + 64) // bt) + 1 + (-(-2 * tiers[t - 1][3] // bt) if t else 0)
        cfg.append(TierConfig(k, v, cap, bt, ring, "host" if case["host"] and t == last else "device",
                              7 + t if case["paged"] else None, t == last and case["select"] > 0))
    cache = TieredCache(B, case["q_heads"], case["kv_heads"], cfg)
    for t in range(last):        # a cache that has been running: the rings of the tiers that evict have moved on
        cache.start[t][:] = [(3 + 7 * b) % cfg[t].ring_blocks * cfg[t].block_tokens for b in range(B)]
    if case["kind"] != "prefill":
        for t in range(last, -1, -1):
            for b, k, v in loads[t]:
                cache.append(t, k, v, seq=b, through_tiers=True)
        loads = None
    return {"case": case, "cache": cache, "q": q, "k": k_new, "v": v_new, "loads": loads,
            "start": [s.copy() for s in cache.start], "len": [n.copy() for n in cache.len]}


def run(state):
    cache, kind = state["cache"], state["case"]["kind"]
    for t in range(len(state["len"])):       # the step, prompt or eviction of this pass starts from the same cache
        cache.start[t][:] = state["start"][t]
        cache.len[t][:] = state["len"][t]
    if kind == "step":
        out, lse = cache.step(state["q"], state["k"], state["v"])
        return out, lse, cache.pool[0]           # the window, with the token's row in it
    if kind == "topk":
        out, lse = cache.step(state["q"], state["k"], state["v"], select_k=state["case"]["select"])
        return out, lse, cache.pool[0], cache.sel_blocks, cache.sel_count
    if kind == "prefill":
        for t in range(len(state["loads"]) - 1, -1, -1):
            for b, k, v in state["loads"][t]:
                cache.append(t, k, v, seq=b, through_tiers=True)
        stored = list(cache.pool)
    else:
        cache.demote()
        stored = list(cache.pool[1:])
    if state["case"]["select"]:
        stored.append(cache.kmu.view(torch.int16))
    return stored, [n.copy() for n in cache.len]


# ------------------------------------------------------------------ the same in 64 bits

def over(x, y):
    """x / y rounded once to 32 bits (a tensor divided by a number is a product with its reciprocal here)."""
    return (x.double() / y).float()


def q1(x):
    g = x.view(*x.shape[:-1], 4, 32)
    s = over(g.abs().amax(-1, keepdim=True), 127.0).half().float()
    c = torch.where(s == 0, torch.zeros_like(g), torch.clamp(torch.round(over(g, s.double())), -127, 127))
    return (c * s).view(x.shape)


def q2(x, dim):
    """Asymmetric 4-bit over the axis `dim` of x."""
    lo, hi = x.amin(dim, keepdim=True), x.amax(dim, keepdim=True)
    s, z = over(hi - lo, 15.0).half().float(), lo.half().float()
    c = torch.where(s == 0, torch.zeros_like(x), torch.clamp(torch.round(over(x - z, s.double())), 0, 15))
    return c * s + z


def stored(x, fmt):
    """fp32 values [heads][tokens][128] as a tier of this format holds them."""
    if fmt == "i8":
        return q1(x)
    if fmt == "i4t":
        return q2(x.view(x.shape[0], -1, 128, 128), 2).view(x.shape)
    if fmt in ("i4", "i4c"):
        return q2(x.view(*x.shape[:-1], 2, 64), -1).view(x.shape)
    return x


def exact(case, seed):
    if case["kind"] in ("prefill", "evict"):
        return None                              # bytes: there is one right answer
    tiers, B, hq, hkv = spec(case), case["batch"], case["q_heads"], case["kv_heads"]
    q, k_new, v_new, loads = inputs(case, seed)
    G, last = hq // hkv, len(tiers) - 1
    out = torch.zeros(B, hq, 128, dtype=torch.float64, device=DEV)
    lse = torch.zeros(B, hq, dtype=torch.float64, device=DEV)
    ids = torch.zeros(B, max(1, case["select"]), dtype=torch.int32)
    count = torch.zeros(B, dtype=torch.int32)
    for b in range(B):
        ks, vs = [k_new[b].float()], [v_new[b].float()]
        for t, (kf, vf, _, bt) in enumerate(tiers):
            k, v = next((x[1][b].float(), x[2][b].float()) if x[0] < 0 else (x[1].float(), x[2].float())
                        for x in loads[t] if x[0] in (-1, b))
            for u in range(1, t):
                k, v = stored(k, tiers[u][0]), stored(v, tiers[u][1])
            if case["kind"] == "topk" and t == last:
                blocks = -(-k.shape[1] // bt)
                pad = torch.zeros(hkv, blocks * bt, 128, device=DEV, dtype=torch.float64)
                pad[:, :k.shape[1]] = k.double()
                mean = (pad.view(hkv, blocks, bt, 128).sum(2) / bt).half().double()
                phi = torch.matmul(mean, q[b].double().view(hkv, G, 128).sum(1).unsqueeze(-1)).squeeze(-1).sum(0)
                keep = torch.sort(torch.topk(phi, min(case["select"], blocks)).indices).values
                ids[b, :len(keep)] = keep.int().cpu()
                count[b] = len(keep)
                tok = (keep.view(-1, 1) * bt + torch.arange(bt, device=DEV)).view(-1)
                tok = tok[tok < k.shape[1]]
                k, v = stored(k, kf)[:, tok], stored(v, vf)[:, tok]
            else:
                k, v = stored(k, kf), stored(v, vf)
            ks.append(k)
            vs.append(v)
        k, v = torch.cat(ks, 1), torch.cat(vs, 1)
        for h in range(hkv):
            s = torch.matmul(q[b, h * G:(h + 1) * G].double(), k[h].double().t().contiguous()) / math.sqrt(128.0)
            lse[b, h * G:(h + 1) * G] = torch.logsumexp(s, -1)
            out[b, h * G:(h + 1) * G] = torch.matmul(torch.softmax(s, -1), v[h].double())
    if case["kind"] == "topk":
        return out, lse, None, ids, count
    return out, lse, None
