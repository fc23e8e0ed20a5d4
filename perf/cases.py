"""Performance cases of the layer-replica library: the calls a serving program
makes on one replica, over the range of sizes it makes them with.

A replica serves its share of a batch: decode steps (one token per request),
prefill chunks (new tokens of a few requests over what they have cached), a
span of layers in one call, and cache appends when requests move to it. Every
case goes through the package's public functions, in place on the hidden
buffer and the paged cache, as a serving loop calls them.

Case fields (all plain values):
  kind    "decode", "prefill" or "append"
  shape   a key of SHAPES
  layers  layers run by the call (more than one: a span)
  rows    decode: requests in the call; prefill / append: new tokens in all
  seqs    prefill / append: requests the tokens belong to
  of      rows of the full-batch hidden buffer the call's rows are picked from
  median, sigma, top   lognormal distribution of the cached context lengths
          (clipped to top); median 0: nothing cached
  lens    seed of the length draws (lengths belong to the case, values to the seed)
  news, priors   explicit lengths instead of drawn ones, comma-separated
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2607_04181_amd as coco

BLOCK = 16

# (d_model, query heads, key/value heads, head_dim, d_ffn, rope theta, eps,
# dtype, longest context a handle of this shape is set up for)
SHAPES = {
    "tiny": (256, 4, 2, 64, 688, 1.0e4, 1e-6, "f32", 1024),
    "small_f32": (1024, 16, 4, 64, 2816, 1.0e4, 1e-6, "f32", 4096),
    "8b": (4096, 32, 8, 128, 14336, 5.0e5, 1e-5, "bf16", 16400),
    "32b": (5120, 40, 8, 128, 27648, 1.0e6, 1e-6, "bf16", 8208),
    "70b": (8192, 64, 8, 128, 28672, 5.0e5, 1e-5, "bf16", 32784),
}


def listed():
    return [
        # The smallest call there is: a tiny fp32 layer, 4 of 8 rows, contexts
        # up to 64 tokens. Launches and latency are all of it.
        dict(name="tiny_decode_4of8", kind="decode", shape="tiny", layers=1, rows=4, of=8,
             median=32, sigma=0.6, top=64, lens=1),
        # fp32 reference runs of a prompt: ragged prefill of a small layer.
        dict(name="f32_prefill_200", kind="prefill", shape="small_f32", layers=1, rows=200,
             seqs=3, of=256, median=150, sigma=0.8, top=1024, lens=2),
        # A replica serving a single request: the layer's weights are the work.
        dict(name="8b_decode_1", kind="decode", shape="8b", layers=1, rows=1, of=1, median=1024,
             sigma=0.1, top=8192, lens=3),
        # The ordinary decode step, batch 64 around 1k tokens of context.
        dict(name="8b_decode_64", kind="decode", shape="8b", layers=1, rows=64, of=64,
             median=1024, sigma=0.8, top=8192, lens=4),
        # A hot replica's uneven share: 96 of 256 in-flight rows, skewed contexts.
        dict(name="8b_decode_96of256", kind="decode", shape="8b", layers=1, rows=96, of=256,
             median=2048, sigma=1.0, top=16384, lens=5),
        # A large decode batch.
        dict(name="8b_decode_256", kind="decode", shape="8b", layers=1, rows=256, of=256,
             median=2048, sigma=1.0, top=16384, lens=6),
        # The 32B-shaped layer's decode step after its chunked prefill.
        dict(name="32b_decode_128", kind="decode", shape="32b", layers=1, rows=128, of=128,
             median=1024, sigma=0.8, top=8192, lens=7),
        # A replicated segment: two 70B-shaped layers in one span call, long contexts.
        dict(name="70b_span2_decode_128", kind="decode", shape="70b", layers=2, rows=128, of=128,
             median=4096, sigma=0.7, top=32768, lens=8),
        # Tails of prompts: a few short ragged requests in one prefill call.
        dict(name="8b_prefill_300", kind="prefill", shape="8b", layers=1, rows=300, seqs=3,
             of=512, news="37,150,113", priors="0,700,2049"),
        # Chunked prefill of 2k tokens over 4 requests with up to 4k cached.
        dict(name="32b_prefill_2048", kind="prefill", shape="32b", layers=1, rows=2048, seqs=4,
             of=2048, news="512,512,512,512", priors="0,512,1024,4096"),
        # A ragged chunk on the largest layer.
        dict(name="70b_prefill_1000", kind="prefill", shape="70b", layers=1, rows=1000, seqs=3,
             of=1024, news="421,512,67", priors="1030,0,4096"),
        # Requests moving to this replica: their cached tokens appended in bulk.
        dict(name="8b_append_6000", kind="append", shape="8b", layers=1, rows=6000, seqs=5,
             news="1733,64,2048,1001,1154", priors="0,128,0,517,33"),
    ]


def draw(rng):
    def log_int(lo, hi):
        return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))

    kind = rng.choice(["decode", "decode", "decode", "prefill", "prefill", "prefill", "append"])
    shape = rng.choice(["8b", "8b", "32b", "70b", "tiny", "small_f32"])
    f32 = SHAPES[shape][7] == "f32"
    c = dict(kind=kind, shape=shape, layers=1, lens=rng.randrange(1 << 30),
             sigma=round(rng.uniform(0.1, 1.0 if shape == "8b" else 0.7), 3))
    if kind == "decode":
        rows = log_int(1, {"8b": 256, "32b": 128, "70b": 128}.get(shape, 256))
        c.update(rows=rows, of=rows + rng.choice([0, rng.randrange(1, 2 * rows + 2)]),
                 median=log_int(16, 256 if f32 else 4096 if shape == "70b" else 2048),
                 top=SHAPES[shape][8] - BLOCK)
        if shape != "70b":
            c["layers"] = rng.choice([1, 1, 2])
    elif kind == "prefill":
        rows = log_int(1, {"8b": 3072, "32b": 2000, "70b": 1000}.get(shape, 512))
        c.update(rows=rows, seqs=min(rows, rng.randrange(1, 9)),
                 of=rows + rng.choice([0, rng.randrange(1, rows + 2)]),
                 median=rng.choice([0, log_int(16, 256 if f32 else 2048)]),
                 top=min(4096, SHAPES[shape][8] // 2))
    else:
        rows = log_int(1, 1024 if f32 else 12000)
        seqs = min(rows, rng.randrange(max(1, -(-rows // (SHAPES[shape][8] // 4))), 13))
        c.update(rows=rows, seqs=seqs, of=1, median=rng.choice([0, log_int(1, 200)]),
                 top=SHAPES[shape][8] // 4)
    return c


# ----------------------------------------------------------------------------
# Lengths (from the case alone)
# ----------------------------------------------------------------------------


def _contexts(rng, n, c):
    if not c["median"]:
        return np.zeros(n, np.int64)
    x = rng.lognormal(math.log(c["median"]), c["sigma"], size=n)
    return np.clip(np.floor(x), 1, c["top"]).astype(np.int64)


def _lengths(c):
    """(cached tokens before the call, new tokens) of each request."""
    if "news" in c:
        return (np.array([int(v) for v in c["priors"].split(",")], np.int64),
                np.array([int(v) for v in c["news"].split(",")], np.int64))
    rng = np.random.default_rng(c["lens"])
    if c["kind"] == "decode":
        return _contexts(rng, c["rows"], c), np.ones(c["rows"], np.int64)
    prior = _contexts(rng, c["seqs"], c)
    # Uneven shares of the new tokens, at least one each, none over the room
    # that the handle's longest context leaves.
    share = rng.uniform(0.2, 1.0, size=c["seqs"])
    room = SHAPES[c["shape"]][8] - prior
    new = np.minimum(1 + np.floor(share / share.sum() * (c["rows"] - c["seqs"])).astype(np.int64),
                     room)
    left = c["rows"] - int(new.sum())
    for s in range(c["seqs"]):
        more = min(left, int(room[s] - new[s]))
        new[s] += more
        left -= more
    assert left == 0, "the new tokens do not fit the contexts"
    return prior, new


# ----------------------------------------------------------------------------
# Inputs
# ----------------------------------------------------------------------------


def _inputs(c, seed):
    d, hq, hkv, hd, ffn, _, _, dtype, longest = SHAPES[c["shape"]]
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(seed)
    rng = np.random.default_rng(seed)

    def normal(*shape, sigma=1.0, mean=0.0):
        t = torch.empty(shape, dtype=dt, device="cuda")
        return t.normal_(mean, sigma, generator=gen)

    def i32(a):
        return torch.from_numpy(np.ascontiguousarray(a, np.int32)).cuda()

    prior, new = _lengths(c)
    n_seqs = len(prior)
    ctx = prior + new
    need = -(-ctx // BLOCK)
    n_blocks = int(need.sum())
    # Physical blocks in shuffled order, as a serving allocator leaves them.
    perm = rng.permutation(n_blocks)
    table = np.full((n_seqs, -(-longest // BLOCK)), -1, np.int64)
    at = 0
    for s, n in enumerate(need):
        table[s, :n] = perm[at:at + n]
        at += n
    positions = np.concatenate([np.arange(p, p + n) for p, n in zip(prior, new)])
    layers = []
    for _ in range(c["layers"]):
        layers.append({
            "w_qkv": normal((hq + 2 * hkv) * hd, d, sigma=0.02),
            "w_o": normal(d, hq * hd, sigma=0.02),
            "w_gate_up": normal(2 * ffn, d, sigma=0.02),
            "w_down": normal(d, ffn, sigma=0.02),
            "gamma_attn": normal(d, sigma=0.1, mean=1.0),
            "gamma_mlp": normal(d, sigma=0.1, mean=1.0),
            "k_cache": normal(n_blocks, hkv, BLOCK * hd),
            "v_cache": normal(n_blocks, hkv, BLOCK * hd),
        })
    st = {"case": c, "layers": layers, "prior": prior, "new": new, "table": table,
          "positions_np": positions, "positions": i32(positions), "block_table": i32(table)}
    if c["kind"] == "append":
        st["k"] = normal(len(positions), hkv, hd)
        st["v"] = normal(len(positions), hkv, hd)
        st["seq_idx"] = i32(np.repeat(np.arange(n_seqs), new))
    else:
        st["hidden"] = normal(c["of"], d)
        st["row_np"] = rng.permutation(c["of"])[:c["rows"]]
        st["row_idx"] = i32(st["row_np"])
        st["ctx_lens"] = i32(ctx)
        st["seq_starts"] = None
        if c["kind"] == "prefill":
            st["seq_starts"] = i32(np.concatenate([[0], np.cumsum(new)]))
    return st


def prepare(case, seed):
    d, hq, hkv, hd, ffn, theta, eps, dtype, longest = SHAPES[case["shape"]]
    st = _inputs(case, seed)
    n_seqs = len(st["prior"])
    # A replica's handle is set up once for the largest call it will get.
    cfg = coco.make_config(d, hq, hkv, hd, ffn, case["layers"], dtype, case["rows"], n_seqs,
                           st["table"].shape[1], theta, eps)
    st["handle"] = coco.coco_layer_init(cfg, st["layers"])
    return st


def run(st):
    c, h = st["case"], st["handle"]
    if c["kind"] == "append":
        coco.coco_kv_append(h, 0, st["k"], st["v"], st["seq_idx"], st["positions"],
                            st["block_table"])
    elif c["layers"] == 1:
        coco.coco_layer_forward(h, 0, st["hidden"], st["row_idx"], st["positions"],
                                st["seq_starts"], st["block_table"], st["ctx_lens"])
    else:
        coco.coco_layer_span_forward(h, 0, c["layers"], st["hidden"], st["row_idx"],
                                     st["positions"], st["seq_starts"], st["block_table"],
                                     st["ctx_lens"])
    out = {"k_cache": [w["k_cache"] for w in st["layers"]],
           "v_cache": [w["v_cache"] for w in st["layers"]]}
    if c["kind"] != "append":
        out["hidden"] = st["hidden"]
    return out


# ----------------------------------------------------------------------------
# Work, tolerance, 64-bit results
# ----------------------------------------------------------------------------


def work(case):
    d, hq, hkv, hd, ffn, _, _, dtype, _ = SHAPES[case["shape"]]
    eb = 2 if dtype == "bf16" else 4
    prior, new = _lengths(case)
    rows = int(new.sum())
    kv_tok = 2 * hkv * hd * eb
    if case["kind"] == "append":
        return {"bytes": rows * (2 * kv_tok + 8), "flops": 0}
    params = d * (hq + 2 * hkv) * hd + d * hq * hd + 3 * d * ffn
    # Keys a row at position p attends: p + 1.
    pairs = int(sum((p + 1 + p + n) * n // 2 for p, n in zip(prior, new)))
    layer_bytes = (params + 2 * d) * eb + int(prior.sum()) * kv_tok + rows * kv_tok
    return {"bytes": case["layers"] * layer_bytes + 2 * rows * d * eb,
            "flops": case["layers"] * (2 * rows * params + 4 * hq * hd * pairs)}


def tolerance(case):
    if case["kind"] == "append":
        return "exact"
    # bf16: q, k, o, h, u are rounded to bf16 between fp32 sums; the rows are
    # 0.003 (batch decode) to 0.009 (prompts without cached context, whose
    # softmax is peaked) off the 64-bit result, by the norm. fp32 differs by
    # the order of its sums: up to 4e-7 for one layer, 5e-7 for two.
    return {"rel": 1.5e-2, "max": 0.3} if SHAPES[case["shape"]][7] == "bf16" else \
        {"rel": 3e-6, "max": 1e-4}


def _k_view(pool, hkv, hd):  # [block, head, dim / 32, dim % 32 / 8, slot, dim % 8]
    return pool.view(-1, hkv, hd // 32, 4, BLOCK, 8)


def _v_view(pool, hkv, hd):  # [block, head, dim / 32, slot / 4, dim % 16, dim % 32 / 16, slot % 4]
    return pool.view(-1, hkv, hd // 32, 4, 16, 2, 4)


def _put(kp, vp, k, v, blk, slot, hkv, hd):
    n = len(blk)
    _k_view(kp, hkv, hd)[blk, :, :, :, slot] = k.view(n, hkv, hd // 32, 4, 8)
    _v_view(vp, hkv, hd)[blk, :, :, slot // 4, :, :, slot % 4] = \
        v.view(n, hkv, hd // 32, 2, 16).transpose(-1, -2)


def _get(kp, vp, blocks, n, hkv, hd):
    """Keys and values of a request's first n tokens, [head, token, dim]."""
    k = _k_view(kp, hkv, hd)[blocks].permute(1, 0, 4, 2, 3, 5).reshape(hkv, -1, hd)[:, :n]
    v = _v_view(vp, hkv, hd)[blocks].permute(1, 0, 3, 6, 2, 5, 4).reshape(hkv, -1, hd)[:, :n]
    return k.double().contiguous(), v.double().contiguous()


def exact(case, seed):
    """The call in 64 bits: plain torch on the same inputs."""
    if case["kind"] == "append":
        return None  # bytes are moved, nothing is computed
    d, hq, hkv, hd, ffn, theta, eps, dtype, _ = SHAPES[case["shape"]]
    st = _inputs(case, seed)
    prior, new, table, pos = st["prior"], st["new"], st["table"], st["positions_np"]
    seq = np.repeat(np.arange(len(prior)), new)
    blk = torch.from_numpy(table[seq, pos // BLOCK]).cuda()
    slot = torch.from_numpy(pos % BLOCK).cuda()
    out = {"k_cache": [], "v_cache": []}
    rows = torch.from_numpy(st["row_np"]).cuda()
    hidden = st["hidden"].double()
    x = hidden[rows]
    inv_freq = theta ** (-2.0 * torch.arange(hd // 2, dtype=torch.float64, device="cuda") / hd)
    angle = torch.from_numpy(pos).cuda().double()[:, None] * inv_freq[None]
    cos, sin = angle.cos()[:, None], angle.sin()[:, None]
    starts = np.concatenate([[0], np.cumsum(new)])
    g = hq // hkv

    def norm(t, gamma):
        return t / torch.sqrt((t * t).mean(-1, keepdim=True) + eps) * gamma.double()

    def rope(t):
        lo, hi = t[..., :hd // 2], t[..., hd // 2:]
        return torch.cat([lo * cos - hi * sin, hi * cos + lo * sin], -1)

    def linear(t, w):
        return torch.nn.functional.linear(t, w.double())

    for w in st["layers"]:
        qkv = linear(norm(x, w["gamma_attn"]), w["w_qkv"]).view(len(pos), hq + 2 * hkv, hd)
        q, k, v = rope(qkv[:, :hq]), rope(qkv[:, hq:hq + hkv]), qkv[:, hq + hkv:].contiguous()
        kp, vp = w.pop("k_cache").double(), w.pop("v_cache").double()
        _put(kp, vp, k, v, blk, slot, hkv, hd)
        o = torch.empty(len(pos), hq, hd, dtype=torch.float64, device="cuda")
        for s in range(len(prior)):
            r0, r1, n = int(starts[s]), int(starts[s + 1]), int(prior[s] + new[s])
            blocks = torch.from_numpy(table[s, :-(-n // BLOCK)]).cuda()
            ks, vs = _get(kp, vp, blocks, n, hkv, hd)
            at = torch.from_numpy(pos[r0:r1]).cuda()
            hidden_key = torch.arange(n, device="cuda")[None] > at[:, None]
            for h in range(hkv):
                qs = q[r0:r1, h * g:(h + 1) * g].transpose(0, 1).reshape(-1, hd)
                z = (qs @ ks[h].T).view(g, r1 - r0, n) / math.sqrt(hd)
                p = z.masked_fill_(hidden_key[None], -math.inf).softmax(-1)
                o[r0:r1, h * g:(h + 1) * g] = \
                    (p.view(-1, n) @ vs[h]).view(g, r1 - r0, hd).transpose(0, 1)
        x = x + linear(o.view(len(pos), hq * hd), w["w_o"])
        gu = linear(norm(x, w["gamma_mlp"]), w["w_gate_up"])
        x = x + linear(torch.nn.functional.silu(gu[:, :ffn]) * gu[:, ffn:], w["w_down"])
        out["k_cache"].append(kp)
        out["v_cache"].append(vp)
    hidden[rows] = x
    out["hidden"] = hidden
    return out
