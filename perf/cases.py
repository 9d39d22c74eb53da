"""The work that a program serving a model with this library has it do, as cases that can be timed.

A case is one of three things: `decode` (one token, or a run of tokens, through the attention of one or more layers),
`stages` (scoring, selection and attention called one by one, as a program does that changes the selected set in
between) and `prefill` (the compression of a layer's prompt, once before its first decode step).  Shapes are those of
sik_workloads.py, the tests and bench.py, and the ranges around them.

Keys of a case: kind; batch, n_kv_heads, n_q_heads; context (tokens resident before the pass), ragged (sequences of
unequal length, from context down to a quarter of it); top_k, per_mille (budget that follows the context), forced
(always-attended tokens per KV head); dtype ("bf16" | "fp16"); cache ("rows": 16-bit K and V, "q2": 2-bit records);
shared (one selection per KV head); append (the new token's key and value join the cache); layers and steps (a pass
takes `steps` tokens through `layers` layers).
"""
import math
import random

import torch

import paper_2603_14224_amd as sik

D = 128
G = D // 4
TORCH = {"bf16": torch.bfloat16, "fp16": torch.float16}


def _case(kind, batch, n_kv_heads, n_q_heads, context, top_k=0, **more):
    c = dict(kind=kind, batch=batch, n_kv_heads=n_kv_heads, n_q_heads=n_q_heads, context=context, top_k=top_k,
             ragged=False, per_mille=0, forced=0, dtype="bf16", cache="rows", shared=False, append=False, layers=1,
             steps=1)
    c.update(more)
    return c


def listed():
    return [
        # the smallest call there is in use: one KV head of a small model, or of a model split over many devices
        dict(_case("decode", 1, 1, 4, 4096, 256, dtype="fp16"), name="decode-4k-one-head"),
        # one user, one token through eight layers of a Llama-3-8B-shaped model at 32K: the library's headline shape
        dict(_case("decode", 1, 8, 32, 32768, 1024, layers=8), name="decode-32k"),
        # one user with a long document: eight tokens through two layers, each appended to the cache
        dict(_case("decode", 1, 8, 32, 131072, 2048, append=True, layers=2, steps=8), name="decode-128k-append"),
        # a server's full batch
        dict(_case("decode", 32, 8, 32, 16384, 512), name="decode-32x16k"),
        # a small batch of long contexts with 8 query heads to a KV head, sixteen tokens generated
        dict(_case("decode", 4, 8, 64, 65536, 1536, append=True, steps=16), name="decode-4x64k-gqa8-append"),
        # a server's ordinary moment: sequences of unequal and odd length, 5 query heads to a KV head (Qwen2.5-14B)
        dict(_case("decode", 7, 8, 40, 12345, 617, ragged=True, dtype="fp16", layers=4), name="decode-ragged-gqa5"),
        # the full batch on the 2-bit cache
        dict(_case("decode", 32, 8, 32, 16384, 512, cache="q2"), name="decode-2bit-32x16k"),
        # the 2-bit cache as the paper runs it: 7.5 % of the context, 64 sink tokens in 16 bits, new tokens appended
        dict(_case("decode", 10, 8, 32, 16384, 1229, cache="q2", per_mille=75, forced=64, append=True, steps=4),
             name="decode-2bit-10x16k-sinks"),
        # one selection for the query heads of a KV head: the cheapest form of the step
        dict(_case("decode", 4, 8, 64, 65536, 1536, shared=True), name="decode-shared-4x64k"),
        # scoring, selection and attention as calls of their own
        dict(_case("stages", 2, 8, 32, 20000, 1000, dtype="fp16"), name="stages-2x20k"),
        # the prompt of one user compressed, keys only
        dict(_case("prefill", 1, 8, 32, 32768), name="prefill-32k-keys"),
        # the prompts of a batch compressed into the 2-bit cache
        dict(_case("prefill", 4, 8, 64, 65536, cache="q2"), name="prefill-4x64k-2bit"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


MOST_KEYS = 32 * 8 * 16384  # keys of a layer in the largest listed batch
MOST_BYTES = 3.7e9          # what the sixteen steps on 4 x 64K move, the most of the listed cases


def draw(rng: random.Random):
    kind = rng.choice(["decode"] * 8 + ["stages"] + ["prefill"] * 3)
    n_kv, n_q = rng.choice([(8, 32), (8, 32), (8, 40), (8, 64), (4, 28), (2, 6), (8, 8), (1, 4)])
    context = _log_uniform(rng, 1024, 131072)
    batch = _log_uniform(rng, 1, 32)
    batch = max(1, min(batch, MOST_KEYS // (n_kv * context)))
    dtype = rng.choice(["bf16", "bf16", "fp16"])
    cache = rng.choice(["rows", "rows", "q2"])
    ragged = batch > 1 and rng.random() < 0.4
    if kind == "prefill":
        return _case(kind, batch, n_kv, n_q, min(context, MOST_KEYS // (2 * batch * n_kv)), ragged=ragged, dtype=dtype,
                     cache=cache)
    top_k = max(32, min(4096, int(context * rng.uniform(0.015, 0.08))))
    if kind == "stages":
        return _case(kind, batch, n_kv, n_q, min(context, MOST_KEYS // (2 * batch * n_kv)), top_k, ragged=ragged,
                     dtype=dtype)
    c = _case(kind, batch, n_kv, n_q, context, top_k, ragged=ragged, dtype=dtype, cache=cache,
              append=rng.random() < 0.5)
    option = rng.choice(["none", "none", "none", "forced", "per_mille", "shared"])
    if option == "forced":
        c.update(forced=64, top_k=max(160, top_k))
    elif option == "per_mille":
        c.update(per_mille=75, top_k=-(-(context + 16) * 75 // 1000))
    elif option == "shared":
        c.update(shared=True)
    steps = rng.choice([1, 4, 8]) if c["append"] else 1
    layers = rng.choice([1, 2, 4])
    one = work(dict(c, steps=1, layers=1))["bytes"]
    if batch * n_kv * context > MOST_KEYS // 4:
        layers = 1
    while steps * layers * one > MOST_BYTES and steps * layers > 1:
        steps, layers = max(1, steps // 2), max(1, layers // 2)
    c.update(steps=steps, layers=layers)
    return c


def _lengths(c):
    """Tokens of each sequence before the pass; unequal ones fall from the context to a quarter of it."""
    B, L = c["batch"], c["context"]
    return [L - (L * 3 * b) // (4 * (B - 1)) if c["ragged"] and B > 1 else L for b in range(B)]


def _budget(c, length):
    k = c["top_k"]
    if c["per_mille"]:
        k = min(k, max(1, -(-length * c["per_mille"] // 1000)))
    return min(k, length)


def work(c):
    B, Hkv, Hq = c["batch"], c["n_kv_heads"], c["n_q_heads"]
    R, lens = Hq // Hkv, _lengths(c)
    keys = Hkv * sum(lens)
    if c["kind"] == "prefill":
        q2 = c["cache"] == "q2"
        # keys (and values) read once; sign codes (and records) written once; means, codebook, counts (and scales)
        small = B * Hkv * (D * 4 + G * 16 * 5 * 4 + (D * 4 if q2 else 0))
        return {"bytes": keys * (D * 2 * (2 if q2 else 1) + D // 8 + (128 if q2 else 0)) + small,
                "flops": keys * D * (12 if q2 else 4)}
    row = 128 if c["cache"] == "q2" else 4 * D
    heads = Hkv if c["shared"] else Hq
    rows = sum(Hkv * min(n, _budget(c, n) * (1 if c["shared"] else R)) for n in lens)
    fixed = B * (Hkv * G * 16 * 4 * 4 + 2 * Hq * D * 2) + (B * Hkv * 4 * D if c["append"] else 0)
    scores = 4 * heads * sum(lens) if c["kind"] == "stages" else 0
    times = c["layers"] * c["steps"]
    return {"bytes": times * (keys * (D // 8) + rows * row + fixed + scores),
            "flops": times * (heads * sum(lens) * G + B * heads * G * 16 * 8 + Hq * 4 * D * sum(_budget(c, n) for n in lens))}


def tolerance(c):
    if c["kind"] == "prefill":
        return {"rel": 1e-5, "differ": 0.0}  # fp32 means, centroids and scales; codes, counts and records as bytes
    # attention comes back in the storage type: half a unit in the last place of bf16 is 4e-3, of fp16 5e-4
    return {"rel": 1e-2 if c["dtype"] == "bf16" else 2e-3, "differ": 0.0}


def _rows(gen, shape, scale, offset, lens, dtype):
    """[B, Hkv, capacity, D] of normal rows with per-channel scale and offset, zero beyond each sequence's length."""
    x = torch.empty(shape, dtype=dtype, device="cuda")
    for b, n in enumerate(lens):
        y = torch.randn(shape[1], shape[2], D, generator=gen, device="cuda")
        x[b] = y.mul_(scale[:, None]).add_(offset[:, None])
        x[b, :, n:] = 0
    return x


def _channels(gen, n_kv):
    """Per (KV head, channel) standard deviation of keys or values: log-normal, with a few outlier channels."""
    s = torch.exp(0.5 * torch.randn(n_kv, D, generator=gen, device="cuda"))
    outlier = torch.rand(n_kv, D, generator=gen, device="cuda").argsort(1)[:, :2]
    return s.scatter(1, outlier, 8 * s.gather(1, outlier))


def prepare(c, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    B, Hkv, Hq, dt, steps = c["batch"], c["n_kv_heads"], c["n_q_heads"], TORCH[c["dtype"]], c["steps"]
    lens, q2 = _lengths(c), c["cache"] == "q2"
    cap = (c["context"] + (steps if c["append"] else 0) + 7) // 8 * 8
    lay = sik.make_layout(B, Hkv, Hq, D, cap, dt, dt)
    start = torch.tensor(lens, dtype=torch.int32, device="cuda")
    s = dict(case=c, layout=lay, workspace=sik.alloc_workspace(lay, c["top_k"]), start=start,
             seq_len=start.repeat(c["layers"], 1).contiguous(), layers=[])
    shape = (B, Hkv, cap, D)
    for li in range(c["layers"]):
        sk, sv = _channels(gen, Hkv), _channels(gen, Hkv)
        off = 0.5 * sk * torch.randn(Hkv, D, generator=gen, device="cuda")
        n = dict(K=_rows(gen, shape, sk, off, lens, dt),
                 V=_rows(gen, shape, sv, torch.zeros_like(off), lens, dt) if c["kind"] != "prefill" or q2 else None,
                 mu=torch.zeros(B, Hkv, D, device="cuda"), codebook=torch.zeros(B, Hkv, G, 16, 4, device="cuda"),
                 counts=torch.zeros(B, Hkv, G, 16, dtype=torch.int32, device="cuda"),
                 codes=torch.zeros(B, Hkv, cap, D // 8, dtype=torch.uint8, device="cuda"),
                 alpha=torch.zeros(B, Hkv, D, device="cuda") if q2 else None,
                 kvq=sik.alloc_kvq(lay) if q2 else None, seq_len=s["seq_len"][li])
        s["layers"].append(n)
        if c["kind"] == "prefill":
            continue
        n["q"] = torch.randn(steps, B, Hq, D, generator=gen, device="cuda").to(dt)
        if c["append"]:
            n["k_new"] = (torch.randn(steps, B, Hkv, D, generator=gen, device="cuda") * sk + off).to(dt)
            n["v_new"] = (torch.randn(steps, B, Hkv, D, generator=gen, device="cuda") * sv).to(dt)
        _compress(s, n)
        if c["forced"]:
            # tokens picked anywhere in the sequence, as a prefill's attention weights would pick them
            w = torch.rand(B, Hkv, cap, generator=gen, device="cuda")
            w.masked_fill_(torch.arange(cap, device="cuda") >= start[:, None, None], -1.0)
            at = w.topk(c["forced"], dim=2).indices
            n["forced"] = at.to(torch.int32).contiguous()
            if q2:
                n["forced_K"], n["forced_V"] = (
                    x.gather(2, at[..., None].expand(-1, -1, -1, D)).contiguous() for x in (n["K"], n["V"]))
        if q2:  # the records stand in for the rows
            n["K"] = n["V"] = None
    if c["kind"] != "prefill":
        s["out"] = torch.zeros(steps, c["layers"], B, Hq, D, dtype=dt, device="cuda")
    if c["kind"] == "stages":
        s["scores"] = torch.zeros(B, Hq, cap, device="cuda")
        s["idx"] = torch.zeros(B, Hq, c["top_k"], dtype=torch.int32, device="cuda")
    return s


def _compress(s, n):
    if n["kvq"] is not None:
        sik.sik_prefill_compress(s["layout"], n["K"], n["V"], n["seq_len"], n["mu"], n["codebook"], n["counts"],
                                 n["codes"], n["alpha"], n["kvq"], s["workspace"])
    else:
        sik.sik_quantize_keys(s["layout"], n["K"], n["seq_len"], 0, 0, sik.SIK_Q_FIT, n["mu"], n["codebook"],
                              n["counts"], n["codes"], s["workspace"])


def _decode(s, n, step, out):
    c, lay, ws = s["case"], s["layout"], s["workspace"]
    q = n["q"][step]
    kn, vn = (n["k_new"][step], n["v_new"][step]) if c["append"] else (None, None)
    if c["forced"] or c["per_mille"] or c["shared"]:
        sik.sik_decode_step_ex(lay, q=q, k_new=kn, v_new=vn, K=n["K"], V=n["V"], kvq=n["kvq"], alpha=n["alpha"],
                               seq_len=n["seq_len"], mu=n["mu"], codebook=n["codebook"], codes=n["codes"],
                               k=c["top_k"], k_per_mille=c["per_mille"], group_shared=c["shared"],
                               forced_idx=n.get("forced"), forced_K=n.get("forced_K"), forced_V=n.get("forced_V"),
                               out=out, workspace=ws)
    elif n["kvq"] is not None:
        sik.sik_decode_step_q2(lay, q, kn, vn, n["kvq"], n["seq_len"], n["mu"], n["alpha"], n["codebook"], n["codes"],
                               c["top_k"], 0.0, out, None, ws)
    else:
        sik.sik_decode_step(lay, q, kn, vn, n["K"], n["V"], n["seq_len"], n["mu"], n["codebook"], n["codes"],
                            c["top_k"], 0.0, out, None, ws)


def run(s):
    c = s["case"]
    if c["kind"] == "prefill":
        n = s["layers"][0]
        _compress(s, n)
        return {k: n[k] for k in ("mu", "codebook", "counts", "codes", "alpha", "kvq")}
    if c["kind"] == "stages":
        n, lay, ws = s["layers"][0], s["layout"], s["workspace"]
        sik.sik_score(lay, n["q"][0], n["codebook"], n["codes"], n["seq_len"], s["scores"])
        sik.sik_topk(lay, s["scores"], n["seq_len"], c["top_k"], s["idx"], ws)
        sik.sik_sparse_attn(lay, n["q"][0], n["K"], n["V"], s["idx"], c["top_k"], 0.0, s["out"][0, 0], ws)
        return {"scores": s["scores"], "out": s["out"]}  # the order inside a row of idx is not specified
    if c["append"]:  # every pass continues the same prompt, as a program that draws several continuations of it
        s["seq_len"].copy_(s["start"].expand_as(s["seq_len"]))
    for step in range(c["steps"]):
        for li, n in enumerate(s["layers"]):
            _decode(s, n, step, s["out"][step, li])
    if not c["append"]:
        return {"out": s["out"]}
    kept = ("codes", "kvq") if c["cache"] == "q2" else ("codes", "K", "V")
    return {"out": s["out"], "seq_len": s["seq_len"], **{k: [n[k] for n in s["layers"]] for k in kept}}
