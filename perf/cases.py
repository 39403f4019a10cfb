"""The calls a serving program makes through the public entry points of this package, as timed
cases: what each prepares, runs, returns and cannot do without.

A turn of an agent routes the user's request over the tool registry (``slb``), splices the chosen
tool's compiled block into the live cache and appends freshly computed tokens (``splice``,
``append``), re-decodes the suffix over the spliced cache (``attn``: one suffix, a whole prefill or
several suffixes in one launch) and then generates token by token (``decode``).  Every case names
one of these kinds and its sizes; ``listed`` holds one to three of each kind, ``draw`` spreads over
the same kinds and ranges.
"""

import math
import random

import torch

from paper_2608_20397_amd import nexus

PAGE = 16

# Attention geometries: (query heads, KV heads, head_dim, rope base, transposed V, soft cap).
GEOMETRIES = {
    "qwen14b": (40, 8, 128, 1e6, False, 0.0),       # Qwen2.5-14B attention shapes
    "gemma": (16, 8, 256, 1e4, True, 50.0),         # soft-capped, token-innermost V cache
    "d64": (32, 8, 64, 1e6, False, 0.0),            # a small model's heads
    "d64wide": (64, 2, 64, 1e6, False, 0.0),        # 32 query heads per KV head
    "d128vt": (40, 8, 128, 1e6, True, 0.0),         # transposed V without a cap
    "d256": (16, 8, 256, 1e4, False, 50.0),         # capped, row-major V
    "tiny": (4, 1, 64, 1e4, False, 0.0),            # the smallest configuration's heads
}


def listed():
    return [
        # one user turn: quantise its embedding and look up the paper's 250-tool registry
        dict(name="slb_turn", kind="slb", n_tools=250, n_queries=1, dim=768, k=3),
        # a routing service's batch over a large registry, eight candidates for the reranker
        dict(name="slb_batch", kind="slb", n_tools=65536, n_queries=256, dim=768, k=8),
        # a 1024-token compiled block spliced and re-anchored in one pass, all 48 layers
        dict(name="splice_block", kind="splice", geom="qwen14b", dtype="bf16", layers=48,
             n_tokens=1024, offset=2043, capacity=3136, interleaved=False),
        # a 512-token redecoded tail appended to a transposed-V cache, 26 layers
        dict(name="append_vt", kind="append", geom="gemma", dtype="bf16", layers=26,
             n_tokens=512, offset=1031, capacity=1600, interleaved=False),
        # the re-decoded tail of a 512-token block and a short user turn at depth 2048
        dict(name="attn_short", kind="attn", geom="qwen14b", dtype="bf16", n_seqs=1, n_s=192,
             n_past=2432, capacity=2624, shuffled=False),
        # full repair of a 1024-token block and its user turn at depth 16384
        dict(name="attn_deep", kind="attn", geom="qwen14b", dtype="bf16", n_seqs=1, n_s=1088,
             n_past=16384, capacity=17472, shuffled=False),
        # 16 blocks spliced all over a shuffled 32K context, their tails re-decoded in one launch
        dict(name="attn_blocks", kind="attn", geom="qwen14b", dtype="bf16", n_seqs=16, n_s=256,
             n_past=0, capacity=32768, shuffled=True),
        # soft-capped suffix over a transposed V cache
        dict(name="attn_softcap", kind="attn", geom="gemma", dtype="bf16", n_seqs=1, n_s=512,
             n_past=8704, capacity=9216, shuffled=False),
        # the prefill of a 4096-token prompt, small-model heads, pages as a server hands them out
        dict(name="prefill_d64", kind="attn", geom="d64", dtype="bf16", n_seqs=1, n_s=4096,
             n_past=0, capacity=4096, shuffled=True),
        # an fp32 cache (the precision a deployment is checked against), a short suffix
        dict(name="attn_f32", kind="attn", geom="qwen14b", dtype="f32", n_seqs=1, n_s=96,
             n_past=1024, capacity=1120, shuffled=False),
        # generation in one long session
        dict(name="decode_one", kind="decode", geom="qwen14b", dtype="bf16", n_seqs=1,
             max_len=17473, min_len=17473, shared=0),
        # generation in 32 sessions over one warm 16384-token prefix
        dict(name="decode_shared", kind="decode", geom="qwen14b", dtype="bf16", n_seqs=32,
             max_len=17473, min_len=16385, shared=16384),
    ]


def _log_int(rng, lo, hi):
    """An integer of [lo, hi], uniform over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.5)))))))


def _draw_kind(rng, kind):
    if kind == "slb":
        return dict(kind=kind, n_tools=_log_int(rng, 1, 65536), n_queries=_log_int(rng, 1, 256),
                    dim=64 * rng.randint(1, 16), k=rng.randint(1, 8))
    if kind in ("splice", "append"):
        geom = rng.choice(["qwen14b", "gemma", "d64", "d128vt", "d256", "tiny"])
        n = _log_int(rng, 1, 1088)
        offset = rng.randint(0, 2048)
        # a transposed fp32 V of head_dim 256 is refused by the splice
        dtype = "bf16" if geom == "gemma" else rng.choice(["bf16", "bf16", "bf16", "f32"])
        return dict(kind=kind, geom=geom, dtype=dtype,
                    layers=_log_int(rng, 1, 48), n_tokens=n, offset=offset,
                    capacity=(offset + n + PAGE - 1) // PAGE * PAGE + PAGE * rng.randint(0, 4),
                    interleaved=rng.random() < 0.25)
    if kind == "attn":
        form = rng.choice(["suffix", "suffix", "prefill", "blocks"])
        dtype = "f32" if rng.random() < 0.2 else "bf16"
        geom = rng.choice(["qwen14b", "qwen14b", "gemma", "d64", "d64wide", "d128vt", "d256",
                           "tiny"])
        if form == "blocks":
            n_seqs = rng.randint(2, 32)
            capacity = 448 * 32 if dtype == "bf16" else 32 * 48
            n_s = _log_int(rng, 1, capacity // 32 - 128) if dtype == "bf16" else \
                _log_int(rng, 1, 8)
            return dict(kind=kind, geom=geom, dtype=dtype, n_seqs=n_seqs, n_s=n_s, n_past=0,
                        capacity=capacity, shuffled=rng.random() < 0.5)
        if form == "prefill":
            n_past, n_s = 0, _log_int(rng, 16, 4096 if dtype == "bf16" else 256)
        else:
            n_past = _log_int(rng, 16, 16384 if dtype == "bf16" else 2048)
            n_s = _log_int(rng, 1, 1088 if dtype == "bf16" else 96)
        return dict(kind=kind, geom=geom, dtype=dtype, n_seqs=1, n_s=n_s, n_past=n_past,
                    capacity=(n_past + n_s + PAGE - 1) // PAGE * PAGE,
                    shuffled=rng.random() < 0.5)
    n_seqs = _log_int(rng, 1, 48)
    max_len = _log_int(rng, 64, 17473)
    min_len = rng.randint(max_len // 2, max_len)
    return dict(kind="decode", geom=rng.choice(["qwen14b", "qwen14b", "gemma", "d64", "d64wide",
                                                "d128vt", "d256"]),
                dtype="bf16", n_seqs=n_seqs, max_len=max_len, min_len=min_len,
                shared=rng.choice([0, min_len // 4, min_len]))


def draw(rng):
    kind = rng.choice(["slb", "splice", "append", "attn", "attn", "attn", "decode", "decode"])
    top = [work(c) for c in listed() if c["kind"] == kind]
    while True:
        case = _draw_kind(rng, kind)
        # fp32 attention is bounded by its own listed case, the rest by the largest of the kind
        if case.get("dtype") == "f32" and kind == "attn":
            ref = [work(c) for c in listed() if c.get("dtype") == "f32" and c["kind"] == kind]
        else:
            ref = top
        w = work(case)
        if all(w[f] <= max(r[f] for r in ref) for f in ("bytes", "flops")):
            return case


def _dtype(case):
    return torch.float32 if case.get("dtype") == "f32" else torch.bfloat16


def _suffixes(case):
    """(lengths, n_past) of an attention case's sequences: several suffixes lie at the ends of
    non-overlapping blocks placed, as a program finds them, at uneven offsets of the context."""
    n = case["n_seqs"]
    if n == 1:
        return [case["n_s"]], [case["n_past"]]
    r = random.Random(1000003 * n + case["n_s"])
    block = case["n_s"] + 128 if case["dtype"] == "bf16" else case["n_s"] + 16
    room = case["capacity"] - n * block
    starts = sorted(r.randint(0, room) for _ in range(n))
    return [case["n_s"]] * n, [s + b * block + block - case["n_s"] for b, s in enumerate(starts)]


def _decode_lens(case):
    r = random.Random(7919 * case["n_seqs"] + case["max_len"])
    lens = [r.randint(case["min_len"], case["max_len"]) for _ in range(case["n_seqs"])]
    lens[r.randrange(len(lens))] = case["max_len"]
    return lens


def work(case):
    kind = case["kind"]
    if kind == "slb":
        n, q, d = case["n_tools"], case["n_queries"], case["dim"]
        return dict(bytes=n * (d + 4) + q * (4 * d + d + 4 + case["k"] * 8 + 8),
                    flops=2 * n * q * d)
    hq, hkv, d = GEOMETRIES[case["geom"]][:3]
    es = 4 if case["dtype"] == "f32" else 2
    if kind in ("splice", "append"):
        elems = case["layers"] * case["n_tokens"] * hkv * d
        return dict(bytes=4 * elems * es, flops=3 * elems)
    if kind == "attn":
        lens, past = _suffixes(case)
        triples = sum(n * p + n * (n + 1) // 2 for n, p in zip(lens, past))
        keys = max(p + n for n, p in zip(lens, past))
        return dict(bytes=2 * es * (sum(lens) * hq * d + keys * hkv * d),
                    flops=4 * d * hq * triples)
    lens = _decode_lens(case)
    shared = min(case["shared"], min(lens)) // PAGE * PAGE
    keys = shared + sum(n - shared for n in lens)
    return dict(bytes=2 * es * (len(lens) * hq * d + keys * hkv * d),
                flops=4 * d * hq * sum(lens))


def tolerance(case):
    if case["kind"] == "slb":
        return "exact"
    if case["kind"] in ("splice", "append"):
        # keys are rounded once to the storage type (9.4e-4 from 64 bits over the whole cache);
        # values move bit for bit
        return {"rel": 4e-3, "max": 1e-2} if case["dtype"] == "bf16" else {"rel": 1e-6,
                                                                          "max": 1e-5}
    # from 64 bits: 1.7e-3 to 2.2e-3 in bf16 (the rounded probabilities and the output), 1.1e-6
    # in fp32
    return {"rel": 9e-3} if case["dtype"] == "bf16" else {"rel": 5e-6}


# ---- inputs: drawn on the device from the seed alone


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(20397 + 7919 * int(seed))
    return g


def _normal(g, shape, std, dtype):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).mul_(std).to(dtype)


def _perm(g, n, shuffled):
    p = torch.randperm(n, generator=g, device="cuda") if shuffled \
        else torch.arange(n, device="cuda")
    return p.to(torch.int32)


def _cache(case, g, layers, n_pages):
    """K and V pools: keys spread so that scaled logits have a standard deviation near 2, as
    trained heads show, values of unit variance."""
    hq, hkv, d, base, vt, cap = GEOMETRIES[case["geom"]]
    dt = _dtype(case)
    k = _normal(g, (layers, n_pages, hkv, PAGE, d), 2.0, dt)
    v = _normal(g, (layers, hkv, d, n_pages * PAGE) if vt
                else (layers, n_pages, hkv, PAGE, d), 1.0, dt)
    return k, v


def _slb_inputs(case, seed):
    """Unit tool vectors; each query mixes two of them with noise, so that the top-two margin
    falls on both sides of the gate."""
    g = _gen(seed)
    n, q, d = case["n_tools"], case["n_queries"], case["dim"]
    tools = torch.nn.functional.normalize(_normal(g, (n, d), 1.0, torch.float32), dim=1)
    a = torch.randint(n, (q,), generator=g, device="cuda")
    b = torch.randint(n, (q,), generator=g, device="cuda")
    w = 0.9 + 0.2 * torch.rand((q, 1), generator=g, device="cuda")
    x = tools[a] + w * tools[b] + _normal(g, (q, d), 0.3 / math.sqrt(d), torch.float32)
    return tools, torch.nn.functional.normalize(x, dim=1).contiguous()


def _kv_inputs(case, seed):
    hq, hkv, d, base, vt, cap = GEOMETRIES[case["geom"]]
    g = _gen(seed)
    n_pages = case["capacity"] // PAGE
    k, v = _cache(case, g, case["layers"], n_pages)
    pm = _perm(g, n_pages, True)
    shape = (case["layers"], case["n_tokens"], hkv, d)
    return k, v, pm, _normal(g, shape, 2.0, _dtype(case)), _normal(g, shape, 1.0, _dtype(case))


def _attn_inputs(case, seed):
    hq, hkv, d, base, vt, cap = GEOMETRIES[case["geom"]]
    g = _gen(seed)
    n_pages = (case["capacity"] + PAGE - 1) // PAGE
    k, v = _cache(case, g, 1, n_pages)
    pm = _perm(g, n_pages, case["shuffled"])
    lens, past = _suffixes(case)
    return k, v, pm, _normal(g, (sum(lens), hq, d), 1.0, _dtype(case)), lens, past


def _decode_inputs(case, seed):
    hq, hkv, d, base, vt, cap = GEOMETRIES[case["geom"]]
    g = _gen(seed)
    lens = _decode_lens(case)
    stride = (max(lens) + PAGE - 1) // PAGE
    sh = min(case["shared"], min(lens)) // PAGE
    private = [(n + PAGE - 1) // PAGE - sh for n in lens]
    n_pages = sh + sum(private)
    k, v = _cache(case, g, 1, n_pages)
    order = _perm(g, n_pages, True)
    maps = torch.zeros((len(lens), stride), dtype=torch.int32, device="cuda")
    nxt = sh
    for b, p in enumerate(private):
        maps[b, :sh] = order[:sh]
        maps[b, sh:sh + p] = order[nxt:nxt + p]
        nxt += p
    q = _normal(g, (len(lens), hq, d), 1.0, _dtype(case))
    return k, v, maps, torch.tensor(lens, dtype=torch.int32, device="cuda"), q, lens


def _paged(case, k, v, pm):
    hq, hkv, d, base, vt, cap = GEOMETRIES[case["geom"]]
    return nexus.PagedKVCache(
        k, v, pm, base, nexus.V_TRANSPOSED if vt else nexus.V_ROWMAJOR,
        nexus.ROPE_INTERLEAVED if case.get("interleaved") else nexus.ROPE_NEOX)


def prepare(case, seed):
    kind = case["kind"]
    s = dict(case=case)
    if kind == "slb":
        tools, s["x"] = _slb_inputs(case, seed)
        s["tools"], s["tool_scale"] = nexus.slb_quantize(tools)       # the registry, offline
        return s
    hq, hkv, d, base, vt, cap = GEOMETRIES[case["geom"]]
    if kind in ("splice", "append"):
        k, v, pm, s["k"], s["v"] = _kv_inputs(case, seed)
        s["cache"] = _paged(case, k, v, pm)
        s["block"] = nexus.Block(s["k"], s["v"], 0, base, s["cache"].rope_style)
        return s
    if kind == "attn":
        k, v, pm, s["q"], s["lens"], s["past"] = _attn_inputs(case, seed)
        cache = s["cache"] = _paged(case, k, v, pm)
        s["starts"] = [sum(s["lens"][:b]) for b in range(len(s["lens"]))]
        if case["n_seqs"] == 1:
            n = nexus.suffix_attn_workspace_bytes(cache, s["lens"][0], hq, s["past"][0])
        else:
            n = nexus.suffix_attn_varlen_workspace_bytes(cache, s["starts"], s["lens"], s["past"],
                                                         hq)
    else:
        k, v, s["maps"], s["seq_len"], s["q"], lens = _decode_inputs(case, seed)
        # the pool's own page map is not read by a decode step
        cache = s["cache"] = _paged(case, k, v, torch.arange(k.shape[1], dtype=torch.int32,
                                                             device="cuda"))
        n = nexus.decode_attn_workspace_bytes(cache, len(lens), hq, case["max_len"])
    # scratch that a serving program keeps from call to call
    s["workspace"] = torch.empty(max(n, 1), dtype=torch.uint8, device="cuda")
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "slb":
        codes, scale = nexus.slb_quantize(s["x"])
        return (codes, scale) + tuple(nexus.slb_scan(s["tools"], s["tool_scale"], codes, scale,
                                                     k=case["k"]))
    cache = s["cache"]
    if kind == "splice":
        nexus.splice_rephase_pages(cache, s["block"], case["offset"], case["offset"])
        return cache.k, cache.v
    if kind == "append":
        nexus.rope_append(cache, s["k"], s["v"], case["offset"], case["offset"])
        return cache.k, cache.v
    cap = GEOMETRIES[case["geom"]][5]
    if kind == "attn":
        if case["n_seqs"] == 1:
            return nexus.suffix_attn(s["q"], cache, 0, s["past"][0], softcap=cap,
                                     workspace=s["workspace"])
        return nexus.suffix_attn_varlen(s["q"], s["starts"], s["lens"], s["past"], cache, 0,
                                        softcap=cap, workspace=s["workspace"])
    return nexus.decode_attn(s["q"], cache, s["maps"], s["seq_len"], case["max_len"], 0,
                             softcap=cap, workspace=s["workspace"])


# ---- the same results in 64 bits, in plain torch


def _quantized(x):
    s = x.abs().amax(1) / 127.0
    c = torch.where(s[:, None] > 0, torch.round(x / s[:, None]), torch.zeros_like(x))
    return c.clamp(-127, 127), s


def _exact_slb(case, seed):
    tools, x = _slb_inputs(case, seed)
    tc, ts = _quantized(tools)
    qc, qs = _quantized(x)
    score = (qc.double() @ tc.double().t()) * ts.double() * qs.double()[:, None]
    k, n = case["k"], case["n_tools"]
    top, idx = score.topk(min(max(k, 2), n), dim=1)
    pad = max(k, 2) - top.shape[1]
    top = torch.nn.functional.pad(top, (0, pad), value=-math.inf)
    margin = top[:, 0] - top[:, 1] if n > 1 else torch.full_like(top[:, 0], math.inf)
    # indices of near-equal scores and the gate at its threshold have no 64-bit value
    return qc.to(torch.int8), qs.double(), None, top[:, :k], margin, None


def _rotated(x, pos, base, interleaved):
    """Keys x [L][T][H][D] rotated to positions pos [T] in 64 bits."""
    d = x.shape[-1]
    theta = base ** (-2.0 * torch.arange(d // 2, device="cuda", dtype=torch.float64) / d)
    ang = (pos.double()[:, None] * theta)[None, :, None, :]
    c, s = torch.cos(ang), torch.sin(ang)
    x = x.double()
    if interleaved:
        a, b = x[..., 0::2], x[..., 1::2]
        return torch.stack((a * c - b * s, b * c + a * s), dim=-1).reshape(x.shape)
    a, b = x[..., :d // 2], x[..., d // 2:]
    return torch.cat((a * c - b * s, b * c + a * s), dim=-1)


def _exact_kv(case, seed):
    hq, hkv, d, base, vt, cap = GEOMETRIES[case["geom"]]
    k, v, pm, bk, bv = _kv_inputs(case, seed)
    j = torch.arange(case["n_tokens"], device="cuda")
    pos = case["offset"] + (j if case["kind"] == "append" else torch.zeros_like(j))
    k, v = k.double(), v.double()
    t = case["offset"] + j
    page, slot = pm.long()[t // PAGE], t % PAGE
    k[:, page, :, slot] = _rotated(bk, pos, base, case["interleaved"]).transpose(0, 1)
    if vt:
        v[:, :, :, page * PAGE + slot] = bv.double().permute(0, 2, 3, 1)
    else:
        v[:, page, :, slot] = bv.double().transpose(0, 1)
    return k, v


def _attend(q, keys, values, first_pos, cap):
    """q [n][G][D] over keys, values [T][D] of one KV head, query i at first_pos + i, 64 bits."""
    n, G, d = q.shape
    s = (q.double().reshape(n * G, d) @ keys.double().t()) / math.sqrt(d)
    if cap > 0:
        s = cap * torch.tanh(s / cap)
    pos = first_pos + torch.arange(n, device="cuda").repeat_interleave(G)
    s.masked_fill_(torch.arange(keys.shape[0], device="cuda")[None, :] > pos[:, None], -math.inf)
    return (torch.softmax(s, dim=1) @ values.double()).reshape(n, G, d)


def _head(k, v, pages, n, h, vt):
    """Keys and values of the first n tokens of one KV head through a page list."""
    d = k.shape[-1]
    keys = k[0, pages, h].reshape(-1, d)[:n]
    if vt:
        return keys, v[0, h].reshape(d, -1, PAGE)[:, pages].reshape(d, -1)[:, :n].t()
    return keys, v[0, pages, h].reshape(-1, d)[:n]


def exact(case, seed):
    kind = case["kind"]
    if kind == "slb":
        return _exact_slb(case, seed)
    if kind in ("splice", "append"):
        return _exact_kv(case, seed)
    hq, hkv, d, base, vt, cap = GEOMETRIES[case["geom"]]
    G = hq // hkv
    if kind == "attn":
        k, v, pm, q, lens, past = _attn_inputs(case, seed)
        seqs = [(sum(lens[:b]), lens[b], past[b], pm.long()) for b in range(len(lens))]
    else:
        k, v, maps, _, q, lens = _decode_inputs(case, seed)
        seqs = [(b, 1, n - 1, maps[b].long()) for b, n in enumerate(lens)]
    out = torch.empty(q.shape, dtype=torch.float64, device="cuda")
    for q0, n, p0, pages in seqs:
        for h in range(hkv):
            heads = slice(h * G, (h + 1) * G)
            for i in range(0, n, 512):                  # bounds the score matrix
                m = min(512, n - i)
                keys, values = _head(k, v, pages, p0 + i + m, h, vt)
                out[q0 + i:q0 + i + m, heads] = _attend(q[q0 + i:q0 + i + m, heads], keys,
                                                        values, p0 + i, cap)
    return out
