"""The work a program has the Spotlight decode path do, as measurable cases.

Four kinds, each through the package's public entry points:

  step      one decode step of one attention layer (Spotlight.decode_step): the new key is hashed
            into the code cache, the queries are hashed, scored against every cached code, the
            k nearest tokens selected and attended
  hash      spotlight_hash_keys: the code cache built after a prefill, or a chunk of keys appended
  retrieve  spotlight_retrieve_topk alone, for programs that attend with a kernel of their own
  attend    spotlight_sparse_decode alone, over an index list the program brings

Shapes are those of `workload.CONFIGS` (LLaMA-2-7B, LLaMA-3-8B and Qwen2.5-7B attention layers), odd
lengths between them, and the linear hash the paper compares with.  Keys and queries come from two
nearly orthogonal cones, hash weights are N(0, 0.05), as in `workload.py`.  The code caches of the
step and retrieve cases are drawn directly, with a probability of its own for each (head, bit), which
concentrates the distances the way the codes of a cone of keys do.
"""
import math

import torch

import paper_2508_19740_amd as sp

D = 128                 # head dimension
DEVICE = "cuda:0"
TYPES = {"f32": torch.float32, "bf16": torch.bfloat16}


def _step(name, batch, hq, hkv, tokens, bits, hidden, topk, kv="bf16", w="bf16", sink=0, local=0, prepack=True):
    return {"name": name, "kind": "step", "batch": batch, "hq": hq, "hkv": hkv, "tokens": tokens, "bits": bits,
            "hidden": hidden, "topk": topk, "kv": kv, "w": w, "sink": sink, "local": local, "prepack": prepack}


def _hash(name, batch, hkv, rows, first, bits, hidden, kv="bf16", w="bf16"):
    return {"name": name, "kind": "hash", "batch": batch, "hq": hkv, "hkv": hkv, "rows": rows, "first": first,
            "tokens": first + rows, "bits": bits, "hidden": hidden, "topk": 1, "kv": kv, "w": w}


def listed():
    return [
        # one head, 4096 tokens, all binary32: the smallest step, nothing but launches and latency
        _step("step-1head-4k-f32", 1, 1, 1, 4096, 128, 256, 128, kv="f32", w="f32"),
        # a 7B layer without grouped heads at an ordinary 32K context, 2 % kept
        _step("step-32head-32k", 1, 32, 32, 32768, 128, 256, 656),
        # the same layer at 512K tokens: the length the method is quoted at
        _step("step-32head-512k", 1, 32, 32, 524288, 128, 256, 10486),
        # grouped heads, long codes, a serving batch, sink and local windows always kept
        _step("step-gqa4-b16-128k", 16, 32, 8, 131072, 256, 512, 2048, sink=4, local=64),
        # groups of seven, an odd length, hash weights as stored (no packed copy)
        _step("step-gqa7-100k", 1, 28, 4, 100003, 128, 256, 2000, prepack=False),
        # a prompt of 128K tokens has just been prefilled, 32 key-value heads
        _hash("prefill-32head-128k", 1, 32, 131072, 0, 128, 256),
        # the same with grouped heads and 256-bit codes
        _hash("prefill-8head-128k-256b", 1, 8, 131072, 0, 256, 512),
        # binary32 keys and weights, an odd number of rows, as in accuracy studies
        _hash("prefill-4head-10k-f32", 1, 4, 10007, 0, 128, 256, kv="f32", w="f32"),
        # the linear hash sign(xR) at the code length it needs
        _hash("prefill-8head-64k-linear512", 1, 8, 65536, 0, 512, 0),
        # a few tokens at once behind a running cache: speculative decoding, small prompt chunks
        _hash("append-17-b8", 8, 8, 17, 8191, 128, 256),
        # retrieval alone over a million tokens of 512-bit codes
        {"name": "retrieve-8head-1m-512b", "kind": "retrieve", "batch": 1, "hq": 8, "hkv": 8, "tokens": 1048576, "bits": 512,
         "hidden": 1024, "topk": 10486, "kv": "bf16", "w": "bf16", "prepack": True},
        # attention alone over a given index list, binary32 rows
        {"name": "attend-gqa4-64k-f32", "kind": "attend", "batch": 2, "hq": 32, "hkv": 8, "tokens": 65536, "bits": 128,
         "hidden": 256, "topk": 1311, "kv": "f32", "w": "bf16"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step"] * 4 + ["hash"] * 3 + ["retrieve", "attend"])
    hkv, group = rng.choice([(1, 1), (32, 1), (8, 4), (8, 8), (4, 7), (4, 8), (16, 2), (2, 8), (8, 1)])
    batch = rng.choice([1, 1, 1, 2, 4, 8, 16])
    bits, hidden = rng.choice([(128, 256)] * 5 + [(64, 128), (256, 512), (256, 256), (512, 1024), (128, 0), (512, 0)])
    kv = rng.choice(["bf16"] * 4 + ["f32"])
    w = kv if kv == "bf16" else rng.choice(["bf16", "f32"])
    esz = 2 if kv == "bf16" else 4
    if kind == "hash":
        # one token up to a long prompt; no more arithmetic than the largest listed one
        most = int(5e11 / (batch * hkv * 2 * (D * hidden + hidden * bits if hidden else D * bits)))
        rows = _log_int(rng, 2, max(2, min(131072, most)))
        first = rng.choice([0, 0, rng.randrange(1, 20000)])
        c = _hash("", batch, hkv, rows, first, bits, hidden, kv, w)
        del c["name"]
        return c
    # no more codes than 512 MB, K and V than 8 GB, attended rows than 500 MB
    heads = batch * hkv
    most = min(524288, (1 << 29) // (heads * bits // 8), (1 << 33) // (heads * 2 * D * esz))
    tokens = _log_int(rng, 1024, max(1024, most))
    topk = max(20, int(tokens * rng.choice([0.01, 0.02, 0.02, 0.04])))
    topk = max(1, min(topk, tokens, 500_000_000 // (heads * group * 2 * D * esz)))
    c = {"kind": kind, "batch": batch, "hq": hkv * group, "hkv": hkv, "tokens": tokens, "bits": bits, "hidden": hidden,
         "topk": topk, "kv": kv, "w": w}
    if kind != "attend":
        c["prepack"] = rng.random() < 0.7
    if kind == "step":
        c["sink"], c["local"] = rng.choice([(0, 0), (0, 0), (4, 64), (0, 1)])
        if c["sink"] + c["local"] > topk:
            c["sink"] = c["local"] = 0
    return c


# ------------------------------------------------------------------ inputs, from the seed alone
def _normal(g, *shape):
    return torch.randn(*shape, generator=g, device=DEVICE)


def _cone(g, shape, axis, dtype):
    """0.8 axis + N(0, I), in the tensor's own type, without a binary32 copy of a large cache."""
    x = torch.empty(shape, dtype=dtype, device=DEVICE)
    return x.normal_(generator=g).add_((0.8 * axis).to(dtype))


def _weights(g, c):
    t = TYPES[c["w"]]
    if c["hidden"] == 0:     # rotations side by side (the paper's initialisation of the linear hash)
        n = -(-c["bits"] // D)
        r = torch.linalg.qr(torch.randn(c["hkv"], n, D, D, generator=torch.Generator().manual_seed(g.initial_seed())))[0]
        return r.reshape(c["hkv"], n * D, D)[:, :c["bits"]].to(t).contiguous().to(DEVICE), None, None
    return tuple((0.05 * _normal(g, c["hkv"], *s)).to(t).contiguous()
                 for s in ((c["hidden"], D), (c["hidden"],), (c["bits"], c["hidden"])))


def _codes(g, c):
    """Packed codes: in every head a quarter of the bits is set with probability 1/4, a quarter with 3/4, the rest with 1/2."""
    shape = (c["batch"], c["hkv"], c["tokens"], c["bits"] // 32)

    def words(*s):
        return torch.randint(-(1 << 31), 1 << 31, s, generator=g, device=DEVICE, dtype=torch.int32)

    uneven, high = words(shape[0], shape[1], 1, shape[3]), words(shape[0], shape[1], 1, shape[3])   # bits by their probability
    a, b = words(*shape), words(*shape)
    return (a & b & (uneven & ~high)) | ((a | b) & (uneven & high)) | (a & ~uneven)


def _axes(g, c):
    mk = torch.nn.functional.normalize(_normal(g, c["batch"], c["hkv"], D), dim=-1)
    mq = _normal(g, c["batch"], c["hq"], D)
    on = mk.repeat_interleave(c["hq"] // c["hkv"], dim=1)
    mq = torch.nn.functional.normalize(mq - (mq * on).sum(-1, keepdim=True) * on, dim=-1)
    return mk.unsqueeze(2), mq


def _inputs(c, seed):
    g = torch.Generator(device=DEVICE).manual_seed(int(seed) * 1000003 + 17)
    kv, kind = TYPES[c["kv"]], c["kind"]
    cache = (c["batch"], c["hkv"], c["tokens"], D)
    mk, mq = _axes(g, c)
    s = {"weights": _weights(g, c)}
    if kind != "hash":
        s["q"] = _cone(g, (c["batch"], c["hq"], D), mq, kv)
    if kind != "retrieve":
        s["K"] = _cone(g, cache, mk, kv)
    if kind in ("step", "attend"):
        s["V"] = torch.empty(cache, dtype=kv, device=DEVICE).normal_(generator=g)
    if kind in ("step", "retrieve"):
        s["codes"] = _codes(g, c)
    if kind == "hash":
        s["codes"] = torch.zeros(c["batch"], c["hkv"], c["tokens"], c["bits"] // 32, dtype=torch.int32, device=DEVICE)
    if kind == "attend":   # one increasing index in each of k equal stretches of the cache
        at = torch.arange(c["topk"], device=DEVICE, dtype=torch.float64) * (c["tokens"] / c["topk"])
        jitter = torch.rand(c["batch"], c["hq"], c["topk"], generator=g, device=DEVICE, dtype=torch.float64)
        idx = (at + jitter * (c["tokens"] / c["topk"])).long().clamp_(max=c["tokens"] - 1)
        s["idx"] = idx.to(torch.int32)
    return s


def prepare(case, seed):
    c = case
    s = _inputs(c, seed)
    s["case"] = c
    # one context per layer, as a model holds them; weights that stay put are packed once
    s["ctx"] = sp.Spotlight(c["batch"], c["hq"], c["hkv"], c["bits"], c["hidden"], c["tokens"], c["topk"],
                            kv_dtype=TYPES[c["kv"]], weight_dtype=TYPES[c["w"]], device=DEVICE)
    if c.get("prepack"):
        s["ctx"].prepack_weights(*s["weights"])
    if c["kind"] in ("step", "retrieve"):
        s["out_idx"] = torch.empty(c["batch"], c["hq"], c["topk"], dtype=torch.int32, device=DEVICE)
    if c["kind"] in ("step", "attend"):
        s["out"] = torch.empty(c["batch"], c["hq"], D, dtype=torch.float32, device=DEVICE)
    return s


def run(state):
    s, c = state, state["case"]
    ctx, kind = s["ctx"], c["kind"]
    if kind == "step":
        ctx.decode_step(s["q"], s["K"], s["V"], *s["weights"], s["codes"], c["tokens"], c["topk"], c["sink"], c["local"],
                        out_idx=s["out_idx"], out=s["out"])
        return {"idx": s["out_idx"], "out": s["out"], "codes": s["codes"]}
    if kind == "hash":
        return {"codes": ctx.hash_keys(s["K"], *s["weights"], c["first"], c["rows"], s["codes"])}
    if kind == "retrieve":
        return {"idx": ctx.retrieve_topk(s["q"], *s["weights"], s["codes"], c["tokens"], c["topk"], out_idx=s["out_idx"])}
    return {"out": ctx.sparse_decode(s["q"], s["K"], s["V"], s["idx"], out=s["out"])}


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    c = case
    esz, wsz = (2 if c["kv"] == "bf16" else 4), (2 if c["w"] == "bf16" else 4)
    kvh, qh = c["batch"] * c["hkv"], c["batch"] * c["hq"]
    mlp = D * c["hidden"] + c["hidden"] * c["bits"] if c["hidden"] else D * c["bits"]
    weights = c["hkv"] * (mlp + c["hidden"]) * wsz
    kind = c["kind"]
    if kind == "hash":
        keys = kvh * c["rows"]
        return {"bytes": keys * (D * esz + c["bits"] // 8) + weights, "flops": 2 * keys * mlp}
    codes = kvh * c["tokens"] * c["bits"] // 8
    rows = min(qh * c["topk"], kvh * c["tokens"])    # heads of a group may share rows
    attend = {"bytes": 2 * rows * D * esz + qh * c["topk"] * 4 + qh * D * (esz + 4), "flops": 4 * qh * c["topk"] * D}
    if kind == "attend":
        return attend
    retrieve = {"bytes": codes + weights + qh * (D * esz + c["topk"] * 4), "flops": 2 * qh * mlp}
    if kind == "retrieve":
        return retrieve
    return {"bytes": retrieve["bytes"] + 2 * rows * D * esz + qh * D * 4 + kvh * (D * esz + c["bits"] // 8),
            "flops": retrieve["flops"] + attend["flops"] + 2 * kvh * mlp}


def tolerance(case):
    # codes and indices are whole numbers and always the same; attention accumulates in binary32
    # (2e-7 from 64 bits at every listed size)
    if case["kind"] in ("hash", "retrieve"):
        return "exact"
    return {"rel": 1e-6, "max": 1e-5, "differ": 0.0}


# ------------------------------------------------------------------ the same in 64 bits, in plain torch
def _hash64(x, weights, group):
    """Code bits [..., L] of x [B, H, D]."""
    w1, b1, w2 = [None if t is None else t.double().repeat_interleave(group, dim=0) for t in weights]
    h = torch.matmul(w1, x.double().unsqueeze(-1)).squeeze(-1)
    if w2 is not None:
        h = h + b1
        h = torch.matmul(w2, (h * torch.sigmoid(h)).unsqueeze(-1)).squeeze(-1)
    return h > 0


def _pack(bits):
    """Hash output c * W + j of a vector is bit 31 - c of word j."""
    b = bits.reshape(*bits.shape[:-1], 32, -1).long()
    shift = torch.arange(31, -1, -1, device=b.device).view(32, 1)
    words = (b << shift).sum(-2)
    return torch.where(words >= 1 << 31, words - (1 << 32), words).int()


def _popcount(x):
    x = x.long() & 0xFFFFFFFF
    x = x - ((x >> 1) & 0x55555555)
    x = (x & 0x33333333) + ((x >> 2) & 0x33333333)
    x = (x + (x >> 4)) & 0x0F0F0F0F
    return ((x * 0x01010101) & 0xFFFFFFFF) >> 24


def exact(case, seed):
    c = case
    if c["kind"] in ("hash", "retrieve"):     # whole numbers only
        return None
    s = _inputs(c, seed)
    group, n, k = c["hq"] // c["hkv"], c["tokens"], c["topk"]
    out = torch.empty(c["batch"], c["hq"], D, dtype=torch.float64, device=DEVICE)
    if c["kind"] == "step":
        s["codes"][:, :, n - 1] = _pack(_hash64(s["K"][:, :, n - 1], s["weights"], 1))
        qcode = _pack(_hash64(s["q"], s["weights"], group))
        t = torch.arange(n, device=DEVICE)
        forced = (t < c["sink"]) | (t >= n - c["local"])
    for b in range(c["batch"]):
        for hq in range(c["hq"]):
            hk = hq // group
            if c["kind"] == "step":
                dist = torch.zeros(n, dtype=torch.long, device=DEVICE)
                for w in range(c["bits"] // 32):
                    dist += _popcount(s["codes"][b, hk, :, w] ^ qcode[b, hq, w])
                order = torch.where(forced, t, (dist + 1) * n + t)
                rows = torch.topk(order, k, largest=False, sorted=False)[1].sort()[0]
            else:
                rows = s["idx"][b, hq].long()
            score = (s["K"][b, hk, rows].double() * s["q"][b, hq].double()).sum(-1) / math.sqrt(D)
            p = torch.softmax(score, 0)
            out[b, hq] = (p.unsqueeze(-1) * s["V"][b, hk, rows].double()).sum(0)
    if c["kind"] == "step":
        return {"idx": None, "out": out, "codes": None}
    return {"out": out}
