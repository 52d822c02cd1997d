"""Performance cases of the multiplexed decoder-layer library.

Each case is one call of a public entry point on the work a serving worker
gives it: a whole layer iteration (`mx_layer_step`), the paged attention on its
own with or without a workspace (`mx_paged_attn`, `mx_paged_attn_static`), and
the cache write of new tokens (`mx_kv_append`).  A batch is `decodes` requests
in the decode phase, with contexts uniform in [ctx_lo, ctx_hi], followed by
`prefill` prompt tokens in `chunks` prefill chunks (ragged when there are
several), the first of which continues a prompt with `cached` tokens already in
the cache.  Pages are drawn from a shuffled pool.
"""
import math

import numpy as np
import torch

import paper_2606_16264_amd as mx

# The benchmark's layer shapes: hidden, ffn, query heads, KV heads, head dim, RoPE base.
SHAPES = {
    "tiny": (256, 1024, 4, 4, 64, 1e4),
    "7b": (4096, 11008, 32, 32, 128, 1e4),
    "13b": (5120, 13824, 40, 40, 128, 1e4),
    "8b": (4096, 14336, 32, 8, 128, 5e5),
    "70b": (8192, 28672, 64, 8, 128, 1e4),
}
EPS = 1e-5
PAGE = 16


def _case(kind, shape, decodes=0, ctx_lo=0, ctx_hi=0, prefill=0, chunks=0, cached=0, name=None):
    c = dict(kind=kind, shape=shape, decodes=decodes, ctx_lo=ctx_lo, ctx_hi=ctx_hi,
             prefill=prefill, chunks=chunks, cached=cached)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: a 256-wide layer, bound by launches and latency (head_dim 64)
        _case("layer", "tiny", 4, 64, 256, 128, 1, 0, "layer tiny mixed"),
        # one interactive user: a single decoding request on a 7B layer
        _case("layer", "7b", 1, 700, 700, name="layer 7b one decode"),
        # a running decode batch with no prefill mixed in
        _case("layer", "7b", 64, 512, 2048, name="layer 7b decode"),
        # the same batch with one prompt chunk piggybacked on it
        _case("layer", "7b", 64, 512, 2048, 512, 1, 0, "layer 7b mixed"),
        # MHA 13B layer: a decode batch and several ragged prompts
        _case("layer", "13b", 128, 32, 1500, 2048, 3, 0, "layer 13b mixed ragged"),
        # GQA 8B layer: large decode batch with the paper's 2048-token chunk
        _case("layer", "8b", 256, 32, 3000, 2048, 1, 0, "layer 8b mixed"),
        # a prompt alone on a prefill worker (time to first token), odd length
        _case("layer", "8b", 0, 0, 0, 1003, 1, 0, "layer 8b prefill"),
        # the largest: a 70B layer with a long chunk beside the decodes
        _case("layer", "70b", 64, 1024, 8192, 8192, 1, 0, "layer 70b mixed"),
        # attention of a decode batch alone, streaming the cache
        _case("attn", "8b", 256, 32, 8192, name="attention 8b decode"),
        # a late chunk of a long prompt: 2048 new tokens over 14336 cached ones
        _case("attn", "8b", 0, 0, 0, 2048, 1, 14336, "attention 8b late chunk"),
        # few requests with long contexts: every decode is split over keys
        _case("attn", "70b", 4, 16000, 32000, name="attention 70b long decodes"),
        # cache write of a prompt chunk's and the decodes' new tokens
        _case("append", "8b", 64, 32, 4096, 4096, 2, 0, "kv append 8b"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["layer"] * 5 + ["attn"] * 3 + ["static", "append"])
    shape = rng.choice(sorted(SHAPES))
    nkv, d = SHAPES[shape][3], SHAPES[shape][4]
    mix = rng.choice(["decode", "mixed", "mixed", "prefill"])
    decodes = lo = hi = prefill = chunks = cached = 0
    if mix != "prefill":
        decodes = _log_int(rng, 1, 256)
        # the cached tokens of all requests take at most about 2 GB
        most = int(min(32768, 2e9 / (decodes * 4 * nkv * d)))
        hi = _log_int(rng, 64, max(65, most))
        lo = rng.randint(max(1, hi // 16), hi)
    if mix != "decode":
        prefill = _log_int(rng, 16, 4096)
        chunks = rng.choice([1, 1, 2, 4])
        cached = rng.choice([0, _log_int(rng, 16, 8192)])
    return _case(kind, shape, decodes, lo, hi, prefill, chunks, cached)


def _requests(case):
    """(phase, n_new, ctx_len) of the requests: the case alone decides them."""
    rng = np.random.default_rng([case["decodes"], case["ctx_lo"], case["ctx_hi"], case["prefill"],
                                 case["chunks"], case["cached"]])
    D, P, C = case["decodes"], case["prefill"], case["chunks"]
    ctx = rng.integers(case["ctx_lo"], case["ctx_hi"] + 1, size=D).tolist() if D else []
    phase, n_new = [mx.MX_DECODE] * D, [1] * D
    if P:
        cuts = sorted(rng.choice(np.arange(1, P), size=C - 1, replace=False).tolist()) if C > 1 else []
        sizes = np.diff([0] + cuts + [P]).tolist()
        phase += [mx.MX_PREFILL] * len(sizes)
        n_new += sizes
        ctx += [case["cached"]] + [0] * (len(sizes) - 1)
    return phase, n_new, ctx


def _inputs(case, seed):
    """Everything of the case that is not this library's own: the batch in plain
    lists, the page tables and the device tensors."""
    H, F, nq, nkv, d, _ = SHAPES[case["shape"]]
    phase, n_new, ctx = _requests(case)
    need = [-(-(c + n) // PAGE) for c, n in zip(ctx, n_new)]
    total = sum(need)
    pool_pages = total + total // 8 + 8
    order = np.random.default_rng(seed).permutation(pool_pages).astype(np.int32)
    at = np.concatenate([[0], np.cumsum(need)])
    pages = [order[at[r]:at[r + 1]].copy() for r in range(len(need))]
    g = torch.Generator(device="cuda").manual_seed(int(seed))

    def normal(*shape, std=1.0):
        t = torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=g)
        return t

    T = sum(n_new)
    s = dict(phase=phase, n_new=n_new, ctx=ctx, pages=pages, pool_pages=pool_pages, T=T)
    # key pages blocked by 32 dims, value pages transposed (the library's pool layout)
    s["k_pool"] = normal(pool_pages, nkv, d // 32, PAGE, 32)
    s["v_pool"] = normal(pool_pages, nkv, d, PAGE)
    if case["kind"] == "layer":
        s["w"] = {"w_qkv": normal((nq + 2 * nkv) * d, H, std=0.02), "w_o": normal(H, nq * d, std=0.02),
                  "w_gu": normal(2 * F, H, std=0.02), "w_down": normal(H, F, std=0.02),
                  "g1": 1 + normal(H, std=0.1), "g2": 1 + normal(H, std=0.1)}
        s["x"] = normal(T, H)
    elif case["kind"] == "append":
        s["k_new"], s["v_new"] = normal(T, nkv, d), normal(T, nkv, d)
    else:
        s["q"] = normal(T, nq, d)
    return s


def prepare(case, seed):
    H, F, nq, nkv, d, theta = SHAPES[case["shape"]]
    s = _inputs(case, seed)
    s["kind"] = case["kind"]
    s["batch"] = mx.Batch(s["phase"], s["n_new"], s["ctx"], s["pages"])
    s["shape"] = mx.attn_shape(nq, nkv, d, s["pool_pages"])
    cfg = None
    if case["kind"] == "layer":
        cfg = s["cfg"] = mx.layer_cfg(H, F, nq, nkv, d, s["pool_pages"], EPS, theta)
        s["packed"] = torch.empty(mx.mx_packed_weights_bytes(cfg), dtype=torch.uint8, device="cuda")
        mx.mx_pack_weights(cfg, s["w"], s["packed"])
        del s["w"]  # a serving program keeps the packed weights only
        s["y"] = torch.empty_like(s["x"])
    elif case["kind"] != "append":
        s["out"] = torch.empty_like(s["q"])
    if case["kind"] != "static":
        n = mx.mx_workspace_bytes_for(s["batch"], s["shape"], cfg)
        s["ws"] = torch.empty(n, dtype=torch.uint8, device="cuda")
    return s


def run(s):
    if s["kind"] == "layer":
        mx.mx_layer_step(s["batch"], s["cfg"], s["packed"], s["x"], s["y"], s["k_pool"],
                         s["v_pool"], s["ws"])
        return {"y": s["y"], "k_pool": s["k_pool"], "v_pool": s["v_pool"]}
    if s["kind"] == "append":
        mx.mx_kv_append(s["batch"], s["shape"], s["k_new"], s["v_new"], s["k_pool"], s["v_pool"],
                        s["ws"])
        return {"k_pool": s["k_pool"], "v_pool": s["v_pool"]}
    if s["kind"] == "attn":
        mx.mx_paged_attn(s["batch"], s["shape"], s["q"], s["k_pool"], s["v_pool"], s["out"], s["ws"])
    else:
        mx.mx_paged_attn_static(s["batch"], s["shape"], s["q"], s["k_pool"], s["v_pool"], s["out"])
    return {"out": s["out"]}


def work(case):
    H, F, nq, nkv, d, _ = SHAPES[case["shape"]]
    _, n_new, ctx = _requests(case)
    T = sum(n_new)
    kv = 2 * nkv * d * 2  # bytes of one token's keys and values
    pairs = sum(n * c + n * (n + 1) // 2 for n, c in zip(n_new, ctx))  # query-key pairs
    if case["kind"] == "append":
        return {"bytes": 2 * T * kv, "flops": 0}
    if case["kind"] != "layer":
        return {"bytes": 2 * T * nq * d * 2 + (sum(ctx) + T) * kv, "flops": 4 * nq * d * pairs}
    params = (nq + 2 * nkv) * d * H + H * nq * d + 3 * F * H
    # x, y, the weights, the cached tokens read and the new ones written
    return {"bytes": 2 * T * H * 2 + 2 * params + sum(ctx) * kv + T * kv,
            "flops": 2 * T * params + 4 * nq * d * pairs}


def tolerance(case):
    if case["kind"] == "append":
        return "exact"  # a byte copy
    # bf16 outputs, measured against the 64-bit reference and taken about four times:
    # attention 0.0024 (one rounding, bf16 probabilities); the layer 0.0023-0.0055
    # (0.0095 at the 70B shape), whose stages each round to bf16
    return {"rel": 2e-2 if case["kind"] == "layer" else 1e-2}


# ------------------------------------------------------------------ 64-bit reference
def _slots(pages, positions):
    p = torch.as_tensor(pages.astype(np.int64), device="cuda")
    pos = torch.as_tensor(positions, device="cuda")
    return p[pos // PAGE], pos % PAGE


def _put(k_pool, v_pool, s, k, v):
    """k, v [T][nkv][d] to the new tokens' slots of the pools (in their layouts)."""
    t = 0
    for r, (n, c) in enumerate(zip(s["n_new"], s["ctx"])):
        page, slot = _slots(s["pages"][r], np.arange(c, c + n))
        kk, vv = k[t:t + n], v[t:t + n]
        k_pool[page, :, :, slot] = kk.reshape(n, kk.shape[1], -1, 32)
        v_pool[page, :, :, slot] = vv
        t += n


def _attention(s, q, k_pool, v_pool):
    """q [T][nq][d] in float64 -> [T][nq * d]."""
    T, nq, d = q.shape
    nkv = k_pool.shape[1]
    out = torch.empty(T, nq, d, dtype=torch.float64, device="cuda")
    t = 0
    for r, (n, c) in enumerate(zip(s["n_new"], s["ctx"])):
        L = c + n
        p = torch.as_tensor(s["pages"][r].astype(np.int64), device="cuda")
        K = k_pool[p].double().permute(1, 0, 3, 2, 4).reshape(nkv, -1, d)[:, :L]
        V = v_pool[p].double().permute(1, 0, 3, 2).reshape(nkv, -1, d)[:, :L]
        mask = torch.arange(L, device="cuda")[None, :] > torch.arange(c, L, device="cuda")[:, None]
        for g in range(nkv):
            hs = slice(g * (nq // nkv), (g + 1) * (nq // nkv))
            sc = torch.matmul(q[t:t + n, hs].permute(1, 0, 2).reshape(-1, d), K[g].t().contiguous())
            sc = (sc / math.sqrt(d)).reshape(-1, n, L).masked_fill_(mask, -math.inf)
            o = torch.matmul(torch.softmax(sc, -1).reshape(-1, L), V[g].contiguous())
            out[t:t + n, hs] = o.reshape(-1, n, d).permute(1, 0, 2)
        t += n
    return out.reshape(T, nq * d)


def _norm(x, g):
    return x / torch.sqrt(x.square().mean(-1, keepdim=True) + EPS) * g


def _linear(x, w):
    return torch.matmul(x, w.double().t())


def exact(case, seed):
    H, F, nq, nkv, d, theta = SHAPES[case["shape"]]
    s = _inputs(case, seed)
    T = s["T"]
    if case["kind"] == "append":
        k_pool, v_pool = s["k_pool"].double(), s["v_pool"].double()
        _put(k_pool, v_pool, s, s["k_new"].double(), s["v_new"].double())
        return {"k_pool": k_pool, "v_pool": v_pool}
    if case["kind"] != "layer":
        return {"out": _attention(s, s["q"].double(), s["k_pool"], s["v_pool"]).reshape(T, nq, d)}
    w = s["w"]
    x = s["x"].double()
    qkv = _linear(_norm(x, w["g1"].double()), w["w_qkv"]).reshape(T, nq + 2 * nkv, d)
    pos = np.concatenate([np.arange(c, c + n) for n, c in zip(s["n_new"], s["ctx"])])
    ang = torch.as_tensor(pos, dtype=torch.float64, device="cuda")[:, None] * torch.as_tensor(
        theta ** (-2.0 * np.arange(d // 2) / d), device="cuda")[None, :]
    cos, sin = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
    lo, hi = qkv[..., :d // 2], qkv[..., d // 2:]
    rot = torch.cat([lo * cos - hi * sin, hi * cos + lo * sin], -1)
    k_pool, v_pool = s["k_pool"].double(), s["v_pool"].double()
    _put(k_pool, v_pool, s, rot[:, nq:nq + nkv], qkv[:, nq + nkv:])
    o = _attention(s, rot[:, :nq], k_pool, v_pool)
    x1 = x + _linear(o, w["w_o"])
    gu = _linear(_norm(x1, w["g2"].double()), w["w_gu"])
    a = torch.nn.functional.silu(gu[:, :F]) * gu[:, F:]
    return {"y": x1 + _linear(a, w["w_down"]), "k_pool": k_pool, "v_pool": v_pool}
