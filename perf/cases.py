"""What a serving program has this library do, as cases that can be timed: decode steps, prefill
steps and whole prompts over paged caches, through the package's public entry points.

Sizes are the configured workloads' (workloads.py: C1-C5 and their E4M3, window, shared-prefix and
whole-prompt variants) and odd sizes of the same ranges.  Values are N(0, 1) rounded to the element
type, slopes 2^(-8(h+1)/Hq), scale 1/sqrt(D), physical blocks a random permutation, as there.
"""
import math
import random

import torch

import paper_2505_02351_amd as G

KV_SCALE = 0.0125           # E4M3 caches of N(0, 1) data: +-448 codes cover +-5.6 sigma
DTYPES = {"f16": torch.float16, "bf16": torch.bfloat16}
DECODE = ("decode", "decode_parts", "decode_e4m3", "decode_window", "decode_shared")
PREFILL = ("prefill_step", "prompt", "prefill_e4m3", "prefill_window")


def _case(kind, dtype, batch, heads, kv_heads, dim, block, ctx, new=(1, 1), alibi=True, part=0, window=0):
    """ctx: range of tokens already cached; new: range of new tokens per sequence."""
    return {"kind": kind, "dtype": dtype, "batch": batch, "heads": heads, "kv_heads": kv_heads, "dim": dim,
            "block": block, "ctx_lo": ctx[0], "ctx_hi": ctx[1], "new_lo": new[0], "new_hi": new[1],
            "alibi": alibi, "part": part, "window": window}


def listed():
    return [
        # one user, a short context: launches and host time are all there is
        dict(_case("decode", "f16", 1, 8, 2, 64, 16, (127, 127)), name="decode_one_short"),
        # a small batch at moderate lengths: start-up against a short stream
        dict(_case("decode", "f16", 16, 32, 8, 128, 16, (255, 2047)), name="decode_batch16"),
        # the headline: a full batch, ragged contexts up to 8k, memory-bound
        dict(_case("decode", "bf16", 64, 32, 4, 128, 32, (1023, 8191)), name="decode_batch64"),
        # few long contexts, the caller fixes the partition size and stores the new rows itself
        dict(_case("decode_parts", "f16", 4, 64, 8, 128, 16, (32767, 32767), part=512), name="decode_long_parts"),
        # the full batch over 8-bit caches
        dict(_case("decode_e4m3", "bf16", 64, 32, 4, 128, 32, (1023, 8191)), name="decode_e4m3_batch64"),
        # local attention (the mask of the path without slopes): the last 1024 tokens
        dict(_case("decode_window", "bf16", 64, 32, 4, 128, 32, (1023, 8191), alibi=False, window=1024),
             name="decode_window1024"),
        # pairs of requests that start with the same prompt
        dict(_case("decode_shared", "bf16", 64, 32, 4, 128, 32, (1023, 8191)), name="decode_shared_pairs"),
        # chunked prefill: 512 new tokens behind 2048 cached ones
        dict(_case("prefill_step", "bf16", 8, 32, 8, 128, 16, (2048, 2048), new=(512, 512)), name="prefill_chunk"),
        # a few short prompts of odd lengths, plain causal attention, head_dim 64
        dict(_case("prompt", "f16", 5, 16, 4, 64, 16, (0, 0), new=(3, 301), alibi=False), name="prompt_short_ragged"),
        # whole prompts, caches filled on the way: the largest call
        dict(_case("prompt", "bf16", 8, 32, 8, 128, 16, (0, 0), new=(2560, 2560)), name="prompt_whole"),
        # ragged chunks over 8-bit caches, plain causal attention
        dict(_case("prefill_e4m3", "bf16", 6, 32, 8, 128, 32, (5, 2999), new=(333, 777), alibi=False),
             name="prefill_e4m3_ragged"),
        # chunked prefill with local attention
        dict(_case("prefill_window", "bf16", 8, 32, 8, 128, 16, (2048, 2048), new=(512, 512), alibi=False, window=512),
             name="prefill_window512"),
    ]


def _log(rng, lo, hi):
    """A whole number, spread over the logarithm of lo .. hi."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))


def draw(rng):
    kind = rng.choice(DECODE + PREFILL)
    heads, kv_heads = rng.choice([(8, 2), (16, 4), (32, 8), (32, 4), (64, 8), (24, 8), (16, 16)])
    if kind == "decode_shared" and heads // kv_heads > 8:
        heads, kv_heads = 32, 4
    dim, block, dtype = rng.choice([64, 128, 128]), rng.choice([16, 32, 64]), rng.choice(["f16", "bf16"])
    alibi = rng.random() < 0.7
    window = _log(rng, 64, 4096) if kind.endswith("window") else 0
    if kind in DECODE:
        batch = _log(rng, 4 if kind == "decode_shared" else 1, 64)
        hi = _log(rng, 100, 32768)
        while batch * hi * kv_heads * dim * 4 > 9e8:                 # bytes of K and V: no more than the headline's range
            batch, hi = max(1, batch * 2 // 3), (hi if batch > 1 else hi * 2 // 3)
        lo = max(1, int(hi * rng.choice([0.1, 0.25, 1.0])))
        part = block * rng.choice([8, 16, 32]) if kind == "decode_parts" else 0
        return _case(kind, dtype, batch, heads, kv_heads, dim, block, (lo, hi), alibi=alibi, part=part, window=window)
    batch = _log(rng, 1, 8)
    new = _log(rng, 8, 2560)
    ctx = 0 if kind == "prompt" else rng.choice([0, _log(rng, 16, 4096)])
    while 4.0 * heads * dim * batch * new * (ctx + new / 2) > 3.5e11:  # no more than the whole prompts
        new = new * 2 // 3
    return _case(kind, dtype, batch, heads, kv_heads, dim, block, (ctx // 3, ctx), new=(max(1, new // 3), new),
                 alibi=alibi, window=window)


def _lengths(case):
    """(cached tokens, new tokens) of each sequence: the case's own, whatever the seed."""
    rng = random.Random("%(batch)d %(ctx_lo)d %(ctx_hi)d %(new_lo)d %(new_hi)d" % case)
    ctx = [rng.randint(case["ctx_lo"], case["ctx_hi"]) for _ in range(case["batch"])]
    new = [rng.randint(case["new_lo"], case["new_hi"]) for _ in range(case["batch"])]
    return ctx, new


def _shared_blocks(case):
    """Blocks that each sequence has in common with the first of its bundle: 90 % of the bundle's
    shortest context."""
    ctx, _ = _lengths(case)
    bundle = 16 // (case["heads"] // case["kv_heads"])
    got = []
    for b in range(case["batch"]):
        b0 = b - b % bundle
        got.append(int(min(ctx[b0:b0 + bundle]) * 0.9) // case["block"] if b != b0 else 0)
    return got


def _scales(case):
    return 1.0 / math.sqrt(case["dim"])


def _slopes(case):
    h = torch.arange(1, case["heads"] + 1, dtype=torch.float64)
    return torch.exp2(-8.0 * h / case["heads"]).float().cuda() if case["alibi"] else None


def prepare(case, seed):
    gen = torch.Generator("cuda").manual_seed(seed)
    cpu = torch.Generator().manual_seed(seed)
    dt, (ctx, new) = DTYPES[case["dtype"]], _lengths(case)
    B, Hq, Hkv, D, bs = case["batch"], case["heads"], case["kv_heads"], case["dim"], case["block"]
    lens = [c + n for c, n in zip(ctx, new)]
    T = sum(new)

    def normal(*shape, dtype=dt):
        return torch.randn(*shape, generator=gen, device="cuda", dtype=torch.float32).to(dtype)

    # the pool: what the batch needs and some blocks of other requests, dealt in random order
    need = [-(-n // bs) for n in lens]
    pool = sum(need) + 16
    order = torch.randperm(pool, generator=cpu).tolist()
    table = torch.zeros(B, max(need), dtype=torch.int32)
    at = 0
    for b in range(B):
        table[b, :need[b]] = torch.tensor(order[at:at + need[b]], dtype=torch.int32)
        at += need[b]
    shared = None
    if case["kind"] == "decode_shared":
        shared = _shared_blocks(case)
        bundle = G.shared_prefix_bundle(Hq, Hkv, D)
        for b in range(B):
            table[b, :shared[b]] = table[b - b % bundle, :shared[b]]
    shape = (pool, Hkv, bs, D)
    if case["kind"].endswith("e4m3"):
        def codes():
            x = torch.randn(shape, generator=gen, device="cuda") * (1.0 / KV_SCALE)
            return x.clamp_(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8)
        k_cache, v_cache = codes(), codes()
    else:
        k_cache, v_cache = normal(*shape), normal(*shape)
    slots = torch.cat([table[b, torch.arange(ctx[b], lens[b]) // bs].long() * bs + torch.arange(ctx[b], lens[b]) % bs
                       for b in range(B)])
    cu = torch.tensor([sum(new[:b]) for b in range(B + 1)], dtype=torch.int32)
    s = {"case": case, "k_cache": k_cache, "v_cache": v_cache, "table": table.cuda(), "slots": slots.cuda(),
         "lens": torch.tensor(lens, dtype=torch.int32).cuda(), "cu": cu.cuda(), "q": normal(T, Hq, D),
         "k": normal(T, Hkv, D), "v": normal(T, Hkv, D), "slopes": _slopes(case), "scale": _scales(case),
         "max_len": max(lens), "max_new": max(new), "ws": None,
         "shared": None if shared is None else torch.tensor(shared, dtype=torch.int32).cuda()}
    s["out"] = torch.empty_like(s["q"])
    if case["kind"] in DECODE:
        if shared is not None:
            n = G.shared_prefix_workspace_bytes(B, Hq, Hkv, D, bs, s["max_len"])
        else:
            how = {"decode": 0, "decode_parts": case["part"]}.get(case["kind"], G.SPLIT_BALANCED)
            n, _ = G.paged_attention_workspace_bytes(B, Hq, Hkv, D, bs, s["max_len"], how)
        if n:
            s["ws"] = torch.empty(n, dtype=torch.uint8, device="cuda")
    return s


def run(s):
    case = s["case"]
    kind, out, q, k, v, kc, vc = case["kind"], s["out"], s["q"], s["k"], s["v"], s["k_cache"], s["v_cache"]
    table, lens, cu, slopes, scale, ws = s["table"], s["lens"], s["cu"], s["slopes"], s["scale"], s["ws"]
    if kind == "decode":
        G.decode_step(out, q, k, v, kc, vc, table, lens, slopes, scale, s["max_len"], ws)
    elif kind == "decode_parts":
        G.reshape_and_cache(k, v, kc, vc, s["slots"])
        G.paged_attention(out, q, kc, vc, table, lens, slopes, scale, s["max_len"], case["part"], ws)
    elif kind == "decode_e4m3":
        G.decode_step_fp8(out, q, k, v, kc, vc, table, lens, slopes, scale, KV_SCALE, KV_SCALE, s["max_len"], ws)
    elif kind == "decode_window":
        G.decode_step_window(out, q, k, v, kc, vc, table, lens, slopes, scale, case["window"], s["max_len"], ws)
    elif kind == "decode_shared":
        G.decode_step_shared(out, q, k, v, kc, vc, table, lens, s["shared"], slopes, scale, s["max_len"], ws)
    elif kind == "prefill_step":
        G.prefill_step(out, q, k, v, kc, vc, table, lens, cu, slopes, scale, s["max_new"])
    elif kind == "prompt":
        G.prompt_prefill(out, q, k, v, kc, vc, table, cu, slopes, scale, s["max_new"])
    elif kind == "prefill_e4m3":
        G.reshape_and_cache_fp8(k, v, kc, vc, s["slots"], KV_SCALE, KV_SCALE)
        G.paged_prefill_fp8(out, q, kc, vc, table, lens, cu, slopes, scale, KV_SCALE, KV_SCALE, s["max_new"])
    else:
        G.reshape_and_cache(k, v, kc, vc, s["slots"])
        G.paged_prefill_window(out, q, kc, vc, table, lens, cu, slopes, scale, case["window"], s["max_new"])
    return {"out": out, "k_cache": kc, "v_cache": vc}


def work(case):
    """Each visible K and V row once per sequence (shared ones once per bundle), the new rows in and
    out, q and the output once; 4 * D operations per (query, visible key, head)."""
    ctx, new = _lengths(case)
    Hq, Hkv, D, W = case["heads"], case["kv_heads"], case["dim"], case["window"]
    kv_bytes = 1 if case["kind"].endswith("e4m3") else 2
    shared = _shared_blocks(case) if case["kind"] == "decode_shared" else [0] * case["batch"]
    rows = pairs = 0
    for c, n, sb in zip(ctx, new, shared):
        rows += (min(c, W - 1) if W else c) - sb * case["block"]
        for i in range(n):
            pairs += min(c + i + 1, W) if W else c + i + 1
    T = sum(new)
    row = Hkv * D
    return {"bytes": 2 * rows * row * kv_bytes + 2 * T * row * (2 + kv_bytes) + 2 * T * Hq * D * 2,
            "flops": 4 * D * Hq * pairs}


def tolerance(case):
    # Errors are those of one rounding of the output to its type (bf16 1.7e-3, f16 2.5e-4 relative in the
    # 2-norm against 64 bits, single elements half an ulp): four times that, and whole values (codes) exact.
    return {"rel": 7e-3, "max": 0.05} if case["dtype"] == "bf16" else {"rel": 1e-3, "max": 0.01}


def exact(case, seed):
    """The attention in 64 bits, sequence by sequence, on plain tensors."""
    s = prepare(case, seed)
    ctx, new = _lengths(case)
    B, Hq, Hkv, D, bs, W = case["batch"], case["heads"], case["kv_heads"], case["dim"], case["block"], case["window"]
    group = Hq // Hkv
    kc, vc, slots = s["k_cache"], s["v_cache"], s["slots"]
    e4m3 = case["kind"].endswith("e4m3")
    for cache, x in ((kc, s["k"]), (vc, s["v"])):
        if e4m3:
            y = (x.float() * (1.0 / torch.tensor(KV_SCALE, dtype=torch.float32)).item()).clamp(-448, 448)
            x = y.to(torch.float8_e4m3fn).view(torch.uint8)
        cache[slots // bs, :, slots % bs] = x

    def rows(cache, b, n):
        j = torch.arange(n, device="cuda")
        x = cache[s["table"][b, j // bs].long(), :, j % bs]              # [n, Hkv, D]
        if e4m3:
            return x.view(torch.float8_e4m3fn).to(torch.float32).double() * float(torch.tensor(KV_SCALE, dtype=torch.float32))
        return x.double()

    out, t = torch.empty(s["q"].shape, dtype=torch.float64, device="cuda"), 0
    scale = float(torch.tensor(s["scale"], dtype=torch.float32))
    for b in range(B):
        n = ctx[b] + new[b]
        k, v = rows(kc, b, n), rows(vc, b, n)
        pos = torch.arange(ctx[b], n, device="cuda").double()[:, None]
        dist = torch.arange(n, device="cuda").double()[None, :] - pos         # [new, n], <= 0 where visible
        hide = (dist > 0) | (dist <= -W) if W else dist > 0
        for h in range(Hq):
            sc = (s["q"][t:t + new[b], h].double() @ k[:, h // group].t().contiguous()) * scale
            if s["slopes"] is not None:
                sc += float(s["slopes"][h]) * dist
            sc.masked_fill_(hide, -math.inf)
            out[t:t + new[b], h] = torch.softmax(sc, dim=1) @ v[:, h // group].contiguous()
        t += new[b]
    return {"out": out, "k_cache": kc, "v_cache": vc}
