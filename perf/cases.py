"""Timed cases: the calls a rollout / serving program makes, over the range of sizes it makes them at.

A case is one pass through the public entry points of ``paper_2605_20863_amd._lib``:

    decode   one decode-attention step (q_tokens > 1: speculative verification)
    shared   the step for GRPO groups whose block tables share prompt blocks
    append   one step's new keys and values written into the paged cache
    step     append + decode attention of every layer of a small batch, captured in a HIP graph
    prefill  causal attention of packed query tokens (chunk 0: every token of every sequence, the
             log-prob forward; otherwise each sequence's last ``chunk`` tokens)

Sequence lengths depend on the case alone (its ``lseed``), so that every seed is the same work; block
tables, queries, caches and scales come from the seed.
"""

import math

import numpy as np
import torch

from paper_2605_20863_amd import _lib

BS = 16  # tokens per cache block
DEV = "cuda"


def _c(name, op, B, hq, hkv, d, kv, median, sigma, lo, hi, **more):
    return dict(name=name, op=op, B=B, hq=hq, hkv=hkv, d=d, kv=kv, median=median, sigma=sigma, lo=lo, hi=hi,
                lseed=more.pop("lseed", 1), **more)


def listed():
    return [
        # smallest: a float32 multi-head step over a few short sequences (the vector kernel)
        _c("decode_mha_f32", "decode", 4, 4, 4, 64, "f32", 0, 0, 1, 256),
        # a few interactive chats, 32 query / 4 KV heads: launches and latency count
        _c("decode_chat_bf16", "decode", 3, 32, 4, 128, "bf16", 700, 0.6, 64, 2048),
        # one serving step of 24 layers replayed from a HIP graph, 8 sequences of about 1k tokens
        _c("step_graph_bf16", "step", 8, 28, 4, 128, "bf16", 1024, 0.5, 64, 4096, layers=24),
        # the step before attention in a large fp8 batch: every slot of a block in turn
        _c("append_fp8", "append", 512, 64, 8, 128, "fp8", 8192, 0.9, 128, 65536),
        # an ordinary rollout batch of a 7B-class model
        _c("decode_7b_bf16", "decode", 64, 28, 4, 128, "bf16", 2048, 0.8, 64, 16384),
        # speculative verification of three drafted tokens on the same batch
        _c("verify4_7b_bf16", "decode", 64, 28, 4, 128, "bf16", 2048, 0.8, 64, 16384, q_tokens=4),
        # GRPO groups of 8 samples over long shared prompts
        _c("shared_grpo_bf16", "shared", 256, 32, 8, 128, "bf16", 1024, 0.8, 1, 8192, samples=8, plo=3072, phi=6144),
        # the largest decode step: 512 long-tailed sequences over an fp8 cache
        _c("decode_fp8", "decode", 512, 64, 8, 128, "fp8", 8192, 0.9, 128, 65536),
        # chunked prefill of one long prompt: its next 512 tokens over 16k cached ones
        _c("chunk_long_bf16", "prefill", 1, 28, 4, 128, "bf16", 0, 0, 16000, 16384, chunk=512),
        # short turns in a serving batch over an fp8 cache: 16 sequences, 64 new tokens each
        _c("chunk_turns_fp8", "prefill", 16, 32, 8, 128, "fp8", 2500, 0.7, 64, 16384, chunk=64),
        # chunked prefill of a whole batch, 512 tokens a sequence
        _c("chunk_batch_bf16", "prefill", 64, 28, 4, 128, "bf16", 2048, 0.8, 64, 16384, chunk=512),
        # the log-prob forward: every token of 64 rollouts
        _c("logprob_bf16", "prefill", 64, 28, 4, 128, "bf16", 2048, 0.8, 64, 16384, chunk=0),
    ]


HEADS = [(28, 4, 128), (32, 4, 128), (64, 4, 128), (32, 8, 128), (64, 8, 128), (8, 1, 128), (16, 4, 64)]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["decode", "decode", "decode", "shared", "append", "step", "prefill", "prefill", "prefill"])
    hq, hkv, d = rng.choice(HEADS)
    kv = rng.choice(["bf16", "bf16", "fp8"])
    sigma = round(rng.uniform(0.2, 0.9), 2)
    lseed = rng.randrange(2, 1 << 30)
    if op == "decode":
        q_tokens = rng.choice([1, 1, 1, 1, 2, 3, 4])
        if q_tokens * (hq // hkv) > 32:
            q_tokens = 1
        if q_tokens == 1 and rng.random() < 0.15:
            kv, hq, hkv, d = "f32", rng.choice([4, 8]), 4, rng.choice([64, 128])
        B = _logint(rng, 1, 512)
        most = 6.0e9 / (B * hkv * 2 * d * {"f32": 4, "bf16": 2, "fp8": 1}[kv])
        median = _logint(rng, 48, max(64, min(16384, most)))
        return _pure(_c("", "decode", B, hq, hkv, d, kv, median, sigma, 1, min(65536, 8 * median), lseed=lseed,
                        q_tokens=q_tokens))
    if op == "shared":
        samples = rng.choice([4, 8, 16])
        plo = _logint(rng, 100, 3000)
        return _pure(_c("", "shared", samples * rng.randint(1, 256 // samples), hq, hkv, d, kv,
                        _logint(rng, 100, 2000), sigma, 1, 8192, lseed=lseed, samples=samples, plo=plo, phi=2 * plo))
    if op == "append":
        return _pure(_c("", "append", _logint(rng, 1, 512), hq, hkv, d, kv, _logint(rng, 48, 8192), sigma, 16, 65536,
                        lseed=lseed))
    if op == "step":
        return _pure(_c("", "step", _logint(rng, 1, 32), hq, hkv, d, "bf16", _logint(rng, 100, 2048), sigma, 16, 4096,
                        lseed=lseed, layers=rng.choice([8, 16, 24])))
    chunk = rng.choice([0, 0, _logint(rng, 8, 2048), _logint(rng, 8, 2048)])
    if chunk:
        B = _logint(rng, 1, 64)
        median = _logint(rng, 128, min(16384, 300000 // B))
    else:  # every token a query: bounded by the flops, which grow with B * median^2
        B = _logint(rng, 1, 64)
        median = _logint(rng, 64, min(8192, math.sqrt(1.5e8 / B)))
    c = _pure(_c("", "prefill", B, hq, hkv, d, kv, median, sigma, 1, min(24576, 8 * median), lseed=lseed, chunk=chunk))
    while work(c)["flops"] > 4e12:  # no dearer than the largest listed one, whatever the lengths came out as
        c["median"] = c["median"] * 3 // 4
    return c


def _pure(c):
    del c["name"]
    return c


# ------------------------------------------------------------------ sizes


def _lengths(c):
    """(sequence lengths, prompt lengths or None), from the case alone."""
    rng = np.random.default_rng(c["lseed"])
    if c["sigma"] > 0:
        x = np.exp(rng.normal(math.log(c["median"]), c["sigma"], size=c["B"]))
        L = np.clip(np.rint(x), c["lo"], c["hi"]).astype(np.int64)
    else:
        L = rng.integers(c["lo"], c["hi"] + 1, size=c["B"])
    if c["op"] != "shared":
        return L, None
    prompts = np.repeat(rng.integers(c["plo"], c["phi"] + 1, size=c["B"] // c["samples"]), c["samples"])
    return prompts + L, prompts


def _counts(c, L):
    return L if c["chunk"] == 0 else np.minimum(L, c["chunk"])


def _esz(kv):
    return {"f32": 4, "bf16": 2, "fp8": 1}[kv]


def work(c):
    """Every cached byte read once (shared blocks once a group), q read and out written once."""
    L, prompts = _lengths(c)
    hq, hkv, d, B = c["hq"], c["hkv"], c["d"], c["B"]
    e, qe = _esz(c["kv"]), 4 if c["kv"] == "f32" else 2
    per_tok = 2 * hkv * d * e
    blocks = int(((L + BS - 1) // BS).sum())
    tok = int(L.sum())
    if c["op"] == "append":
        # new K and V read and written, and the tables
        return {"bytes": B * (2 * hkv * d * (2 + e) + (16 * hkv if c["kv"] == "fp8" else 0) + 8), "flops": 0.0}
    if c["op"] == "prefill":
        n = _counts(c, L)
        seen = int((n * L - n * (n - 1) // 2).sum())
        byt = tok * per_tok + int(n.sum()) * hq * d * 4 + 4 * blocks
        return {"bytes": byt + (8 * hkv * blocks if c["kv"] == "fp8" else 0), "flops": 4.0 * d * hq * seen}
    if c["op"] == "shared":
        once = prompts[:: c["samples"]] // BS * BS
        tok = tok - int((prompts // BS * BS).sum()) + int(once.sum())
    Q = c.get("q_tokens", 1)
    byt = tok * per_tok + 2 * B * Q * hq * d * qe + 4 * blocks + 4 * B
    if c["kv"] == "fp8":
        byt += 8 * hkv * ((tok + BS - 1) // BS)
    layers = c.get("layers", 1)
    if c["op"] == "step":
        byt += 2 * B * hkv * d * 2 * e
    return {"bytes": layers * byt, "flops": layers * 4.0 * d * hq * Q * int(L.sum())}


def tolerance(c):
    if c["op"] == "append":
        return "exact"
    # outputs in the queries' type: measured against 64 bits, 1.4e-7 in float32 and 1.6e-3 to 1.7e-3 in
    # bfloat16 (one rounding of the result; its products keep more); four times that, and a little for longer sums
    return {"rel": 1e-6 if c["kv"] == "f32" else 7e-3}


# ------------------------------------------------------------------ inputs


def _gen(seed, *key):
    s = np.random.SeedSequence(entropy=int(seed), spawn_key=key).generate_state(1, dtype=np.uint64)[0]
    return torch.Generator(device=DEV).manual_seed(int(s & np.uint64((1 << 62) - 1)))


def _randn(shape, dtype, gen):
    return torch.randn(shape, generator=gen, device=DEV, dtype=torch.float32).to(dtype)


def _fill(x, scales, gen):
    """N(0, 1) cache tiles x [NB, hkv, ., .]; an fp8 cache as codes with one amax scale a tile."""
    step = max(1, (1 << 28) // x[0].numel())
    for i in range(0, x.shape[0], step):
        y = torch.randn(x[i:i + step].shape, generator=gen, device=DEV, dtype=torch.float32)
        if scales is None:
            x[i:i + step] = y.to(x.dtype)
        else:
            s = torch.clamp(y.abs().amax(dim=(2, 3)) / 448.0, min=2.0 ** -126)
            scales[i:i + step] = s
            y.div_(s[:, :, None, None]).clamp_(-448.0, 448.0)
            x[i:i + step] = y.to(torch.float8_e4m3fn).view(torch.uint8)


def _table(L, prompts, samples, width, seed):
    """Block table (physical ids: a random permutation, 5% spare) and the number of physical blocks."""
    nblk = (L + BS - 1) // BS
    t = np.zeros((len(L), max(width, int(nblk.max()))), dtype=np.int64)
    used = np.zeros_like(t, dtype=bool)
    n = 0
    for b in range(len(L)):
        s = 0
        if prompts is not None:
            s = int(prompts[b]) // BS
            if b % samples == 0:
                first = n
                n += s
            t[b, :s] = np.arange(first, first + s)
        k = int(nblk[b])
        t[b, s:k] = np.arange(n, n + k - s)
        n += k - s
        used[b, :k] = True
    nb = n + max(1, n // 20)
    perm = np.random.default_rng(seed).permutation(nb)
    return torch.from_numpy(np.where(used, perm[t], -1).astype(np.int32)).to(DEV), nb


def prepare(c, seed):
    B, hq, hkv, d, kv = c["B"], c["hq"], c["hkv"], c["d"], c["kv"]
    L, prompts = _lengths(c)
    dt = {"f32": torch.float32, "bf16": torch.bfloat16, "fp8": torch.uint8}[kv]
    qdt = torch.float32 if kv == "f32" else torch.bfloat16
    layers = c.get("layers", 1)
    width = 0
    if c["op"] == "append":
        # only blocks that this pass's 16 positions touch exist; the tables are as wide as the sequences
        lo = L // BS
        width = int(lo.max()) + 2
        nb = 2 * B + 1
        perm = np.random.default_rng(seed).permutation(nb)
        t = np.full((B, width), -1, dtype=np.int32)
        t[np.arange(B), lo] = perm[:B]
        t[np.arange(B), lo + 1] = perm[B:2 * B]
        table = torch.from_numpy(t).to(DEV)
    else:
        if c["op"] == "step":
            width = c["hi"] // BS  # a captured graph's tables have room for the sequences to grow
        table, nb = _table(L, prompts, c.get("samples", 1), width, seed)
    lead = (layers,) if layers > 1 else ()
    k = torch.empty(lead + (nb, hkv, BS, d), dtype=dt, device=DEV)
    v = torch.empty(lead + (nb, hkv, d, BS), dtype=dt, device=DEV)
    scales = torch.empty((2, nb, hkv), dtype=torch.float32, device=DEV) if kv == "fp8" else None
    _fill(k.view(-1, hkv, BS, d), None if scales is None else scales[0], _gen(seed, 1))
    _fill(v.view(-1, hkv, d, BS), None if scales is None else scales[1], _gen(seed, 2))
    s = dict(case=c, k=k, v=v, scales=scales, table=table, lens=torch.from_numpy(L.astype(np.int32)).to(DEV),
             scale=1.0 / math.sqrt(d))
    if c["op"] in ("append", "step"):
        shape = lead + (B, hkv, d)
        s["k_new"], s["v_new"] = _randn(shape, torch.bfloat16, _gen(seed, 3)), _randn(shape, torch.bfloat16, _gen(seed, 4))
    if c["op"] == "append":
        # decoding goes on: 16 consecutive positions of every sequence, one a pass
        s["pos"] = [torch.from_numpy((L + i).astype(np.int32)).to(DEV) for i in range(BS)]
        s["at"] = 0
        return s
    if c["op"] == "prefill":
        n = _counts(c, L)
        s["offsets"] = torch.from_numpy(np.concatenate([[0], np.cumsum(n)]).astype(np.int32)).to(DEV)
        s["q"] = _randn((int(n.sum()), hq, d), qdt, _gen(seed, 5))
    elif c.get("q_tokens", 1) > 1:
        s["q"] = _randn((B, c["q_tokens"], hq, d), qdt, _gen(seed, 5))
    else:
        s["q"] = _randn(lead + (B, hq, d), qdt, _gen(seed, 5))
    s["out"] = torch.empty_like(s["q"])
    if c["op"] == "shared":
        s["shared"] = torch.from_numpy((prompts[:: c["samples"]] // BS).astype(np.int32)).to(DEV)
    if c["op"] == "step":
        s["pos"] = s["lens"] - 1
        _capture(s)
    return s


def _layer(s, i):
    """Append the new token's key and value to layer i's cache, then attend over it."""
    _lib.paged_kv_append(s["k_new"][i], s["v_new"][i], s["k"][i], s["v"][i], None, s["table"], s["pos"])
    _lib.paged_decode_attention(s["q"][i], s["k"][i], s["v"][i], s["table"], s["lens"], None, s["out"][i], s["scale"])


def _capture(s):
    """All layers' calls of the step in one HIP graph, as a serving loop keeps it."""
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        _layer(s, 0)  # sizes the stream's workspace before the capture
    stream.synchronize()
    s["graph"] = torch.cuda.CUDAGraph()
    s["stream"] = stream
    with torch.cuda.graph(s["graph"], stream=stream):
        for i in range(s["case"]["layers"]):
            _layer(s, i)


def run(s):
    c = s["case"]
    op = c["op"]
    if op == "decode":
        return _lib.paged_decode_attention(s["q"], s["k"], s["v"], s["table"], s["lens"], s["scales"], s["out"],
                                           s["scale"])
    if op == "shared":
        return _lib.paged_decode_attention_shared_prefix(s["q"], s["k"], s["v"], s["table"], s["lens"], s["scales"],
                                                         s["out"], s["scale"], c["samples"], s["shared"])
    if op == "append":
        _lib.paged_kv_append(s["k_new"], s["v_new"], s["k"], s["v"], s["scales"], s["table"], s["pos"][s["at"]])
        s["at"] = (s["at"] + 1) % BS
        return {"k": s["k"], "v": s["v"], "scales": s["scales"]}
    if op == "step":
        s["graph"].replay()
        return {"out": s["out"], "k": s["k"], "v": s["v"]}
    return _lib.paged_prefill_attention(s["q"], s["offsets"], s["k"], s["v"], s["table"], s["lens"], s["scales"],
                                        s["out"], s["scale"])


# ------------------------------------------------------------------ 64-bit results


def _inputs(c, seed):
    """The inputs of prepare(), without the calls that a graph's capture makes."""
    if c["op"] != "step":
        return prepare(c, seed)
    global _capture
    keep, _capture = _capture, lambda s: None
    try:
        return prepare(c, seed)
    finally:
        _capture = keep


def _attend(q, k, v, scale, see):
    """softmax(scale q k^T) v in float64: q [n, hq, d], k, v [L, hkv, d]; row i sees see[i] keys."""
    n, hq, d = q.shape
    L, hkv, _ = k.shape
    out = torch.empty(q.shape, dtype=torch.float64, device=q.device)
    g = hq // hkv
    keys = torch.arange(L, device=q.device)
    rows = max(1, (1 << 27) // max(1, L * g))  # query rows at a time
    for h in range(hkv):
        kt, vh = k[:, h].t().contiguous(), v[:, h].contiguous()
        for i in range(0, n, rows):
            x = q[i:i + rows, h * g:(h + 1) * g].to(torch.float64)
            m = x.shape[0]
            y = (x.reshape(m * g, d) @ kt).view(m, g, L).mul_(scale)
            y.masked_fill_((keys[None, :] >= see[i:i + rows, None])[:, None, :], -math.inf)
            w = torch.softmax(y, dim=-1).view(m * g, L)
            out[i:i + rows, h * g:(h + 1) * g] = (w @ vh).view(m, g, d)
    return out


def _tokens(x, scale, ids, L, is_v):
    """Tokens 0 .. L - 1 of one sequence's tiles, dequantised to float64: [L, hkv, d]."""
    t = x[ids]
    if scale is not None:
        t = t.view(torch.float8_e4m3fn).to(torch.float32).to(torch.float64) * scale[ids].to(torch.float64)[:, :, None, None]
    t = t.to(torch.float64)
    t = t.permute(0, 3, 1, 2) if is_v else t.permute(0, 2, 1, 3)
    return t.reshape(-1, t.shape[2], t.shape[3])[:L]


def _sequence(s, layer, b, L, q, n):
    """Rows q [n, hq, d], the last n tokens of sequence b, over its L cached tokens."""
    k, v = (s["k"], s["v"]) if layer is None else (s["k"][layer], s["v"][layer])
    ids = s["table"][b, : (L + BS - 1) // BS].long()
    ks, vs = (None, None) if s["scales"] is None else s["scales"]
    see = torch.arange(L - n + 1, L + 1, device=q.device)
    return _attend(q, _tokens(k, ks, ids, L, False), _tokens(v, vs, ids, L, True), s["scale"], see)


def exact(c, seed):
    """run()'s attention outputs in float64; an append's outputs are stored codes, with no such value."""
    if c["op"] == "append":
        return None
    s = _inputs(c, seed)
    L, _ = _lengths(c)
    out = torch.empty(s["q"].shape, dtype=torch.float64, device=DEV)
    if c["op"] == "prefill":
        n = _counts(c, L)
        o = np.concatenate([[0], np.cumsum(n)])
        for b in range(c["B"]):
            out[o[b]:o[b + 1]] = _sequence(s, None, b, int(L[b]), s["q"][o[b]:o[b + 1]], int(n[b]))
        return out
    if c["op"] == "step":
        pos = s["pos"].long()
        at = s["table"].gather(1, (pos // BS)[:, None])[:, 0].long()
        s["k"][:, at, :, pos % BS] = s["k_new"].permute(1, 0, 2, 3)
        s["v"][:, at, :, :, pos % BS] = s["v_new"].permute(1, 0, 2, 3)
        for i in range(c["layers"]):
            for b in range(c["B"]):
                out[i, b] = _sequence(s, i, b, int(L[b]), s["q"][i, b][None], 1)[0]
        return {"out": out, "k": None, "v": None}
    for b in range(c["B"]):
        q = s["q"][b]
        rows = q[None] if q.dim() == 2 else q
        out[b] = _sequence(s, None, b, int(L[b]), rows, rows.shape[0]).view(q.shape)
    return out
