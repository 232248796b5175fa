"""The work that a program using this framework has it do, for timing.

Every case goes through the package's public entry points with the layer shapes of `synth.CONFIGS`
(hidden size 2048, 128 or 256 experts, top-8, intermediate size 512 or 768, the small fp32 layer of 256)
and with odd sizes beside them.  `listed()` gives the cases, `draw()` more of the same ranges, `prepare()`
the inputs and handles a program holds before the call, `run()` one pass, `work()` the bytes and
operations that the pass cannot do without, and `exact()` the same outputs in 64 bits from plain torch.
"""
import math

import numpy as np
import torch

import paper_2605_29135_amd as moe

DT = {"f32": moe.MOE_F32, "bf16": moe.MOE_BF16, "int4": moe.MOE_INT4G128}
SIGMA = 0.02       # weights are N(0, 0.02)
MASK = 64.0        # additive router mask that fixes a token's expert set
EPS = 1e-6


def listed():
    return [
        # Routing of one decode token: the smallest call, on the path of every layer of every token.
        {"name": "route_token", "kind": "route", "T": 1, "H": 2048, "E": 128, "k": 8, "dtype": "bf16"},
        # Routing of a prompt chunk of one layer.
        {"name": "route_chunk", "kind": "route", "T": 2048, "H": 2048, "E": 256, "k": 8, "dtype": "bf16"},
        # The expert FFN of one decode token, bf16 experts (the headline workload's layer).
        {"name": "ffn_bf16_token", "kind": "ffn", "T": 1, "H": 2048, "I": 768, "E": 128, "k": 8, "dtype": "bf16",
         "shared": False, "noalloc": False},
        # The same for int4 experts with a shared one, through the call that allocates nothing (serving loops).
        {"name": "ffn_int4_token", "kind": "ffn", "T": 1, "H": 2048, "I": 512, "E": 256, "k": 8, "dtype": "int4",
         "shared": True, "noalloc": True},
        # A decode batch of 16 tokens, bf16 experts and a shared one.
        {"name": "ffn_bf16_batch16", "kind": "ffn", "T": 16, "H": 2048, "I": 512, "E": 256, "k": 8, "dtype": "bf16",
         "shared": True, "noalloc": False},
        # A small odd decode batch (speculative tokens, a few sequences) on int4 experts.
        {"name": "ffn_int4_batch5", "kind": "ffn", "T": 5, "H": 2048, "I": 512, "E": 256, "k": 8, "dtype": "int4",
         "shared": True, "noalloc": False},
        # A ragged fp32 layer (sizes that fill no lane layout), an odd batch.
        {"name": "ffn_f32_ragged", "kind": "ffn", "T": 7, "H": 1408, "I": 384, "E": 60, "k": 4, "dtype": "f32",
         "shared": False, "noalloc": False},
        # The expert FFN of a whole prompt chunk, int4 experts (the prompt side of the int4 workload).
        {"name": "prefill_int4_chunk", "kind": "prefill", "T": 2048, "H": 2048, "I": 512, "E": 256, "k": 8,
         "dtype": "int4", "shared": True, "zipf": False},
        # A short prompt of odd length on bf16 experts, some experts far busier than others.
        {"name": "prefill_bf16_short", "kind": "prefill", "T": 517, "H": 2048, "I": 768, "E": 128, "k": 8,
         "dtype": "bf16", "shared": False, "zipf": True},
        # The self-attention block of one token at the end of a 4096-position cache.
        {"name": "attention_4k", "kind": "attention", "H": 2048, "heads": 32, "kv": 4, "d": 128, "max_pos": 4096,
         "p": 4095},
        # Whole decode steps of a small all-resident stack, one token at a time.
        {"name": "decode_resident", "kind": "decode", "L": 4, "H": 2048, "I": 768, "E": 128, "k": 8, "dtype": "bf16",
         "shared": False, "slots": 0, "tokens": 2},
        # Whole decode steps under a memory budget: slots for a part of the experts, the misses filled over
        # the host link (the purpose of the framework).
        {"name": "decode_budget", "kind": "decode", "L": 6, "H": 2048, "I": 512, "E": 256, "k": 8, "dtype": "int4",
         "shared": True, "slots": 140, "tokens": 8},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["route", "ffn", "ffn", "ffn", "prefill", "prefill", "attention", "decode"])
    if kind == "route":
        dtype = rng.choice(["bf16", "bf16", "f32"])
        E = rng.choice([16, 60, 128, 130, 256, _log(rng, 8, 256)])
        return {"kind": kind, "T": _log(rng, 1, 2048 if dtype == "bf16" else 256),
                "H": 128 * _log(rng, 2, 16), "E": E, "k": rng.randint(1, min(8, E)), "dtype": dtype}
    if kind == "ffn":
        dtype = rng.choice(["bf16", "bf16", "int4", "int4", "f32"])
        E = rng.choice([16, 60, 128, 256, _log(rng, 8, 256)])
        return {"kind": kind, "T": rng.choice([1, 1, 2, 4, 8, 16, rng.randint(2, 16)]), "H": 128 * _log(rng, 2, 16),
                "I": 128 * _log(rng, 1, 4 if dtype == "f32" else 6), "E": E, "k": rng.randint(1, min(8, E)),
                "dtype": dtype, "shared": rng.random() < 0.5, "noalloc": rng.random() < 0.3}
    if kind == "prefill":
        E = rng.choice([16, 60, 128, 256, _log(rng, 8, 256)])
        return {"kind": kind, "T": _log(rng, 17, 2048), "H": 128 * _log(rng, 4, 16), "I": 128 * rng.randint(1, 4),
                "E": E, "k": rng.randint(1, min(8, E)), "dtype": rng.choice(["int4", "bf16"]),
                "shared": rng.random() < 0.5, "zipf": rng.random() < 0.5}
    if kind == "attention":
        kv = rng.choice([1, 2, 4, 8])
        d = rng.choice([64, 128])
        heads = kv * rng.choice([g for g in (1, 2, 4, 8) if 128 <= kv * g * d <= 4096])
        max_pos = _log(rng, 64, 8192)
        return {"kind": kind, "H": 128 * _log(rng, 4, 16), "heads": heads, "kv": kv, "d": d, "max_pos": max_pos,
                "p": max_pos - 1 - rng.randint(0, max_pos // 8)}
    budget = rng.random() < 0.5
    L, tokens, E, k = rng.randint(2, 4), rng.randint(1, 6), rng.choice([32, 64, 100]), rng.randint(2, 8)
    return {"kind": "decode", "L": L, "H": 128 * _log(rng, 4, 16), "I": 128 * rng.randint(1, 4), "E": E, "k": k,
            "dtype": rng.choice(["bf16", "int4"]), "shared": rng.random() < 0.5,
            "slots": max(k, int(L * k * rng.uniform(1.5, 3.0))) if budget else 0, "tokens": tokens}


# ------------------------------------------------------------------------------------------------ inputs ---
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _normal(shape, g, scale=1.0):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).mul_(scale)


def _matrix(n, rows, cols, dtype, g):
    """n weight matrices [rows x cols] as stored: uint8 [n, bytes]."""
    w = _normal((n, rows, cols), g, SIGMA)
    if dtype == "f32":
        return w.view(n, -1).view(torch.uint8)
    if dtype == "bf16":
        return w.to(torch.bfloat16).view(n, -1).view(torch.uint8)
    w = w.view(n, rows, cols // 128, 128)
    s = (w.abs().amax(-1, keepdim=True) / 7.0).to(torch.bfloat16)
    q = torch.clamp(torch.round(w / s.float()), -8, 7).to(torch.int8).view(n, rows * cols // 2, 2)
    nib = (q[..., 0] & 15) | (q[..., 1] << 4)
    return torch.cat([nib.view(torch.uint8), s.reshape(n, -1).view(torch.uint8)], 1)


def _experts(n, H, I, dtype, g):
    """n expert blobs (gate/up, then down), uint8 [n, expert bytes]."""
    out = None
    for i in range(0, n, 32):  # a few at a time: the fp32 draws are larger than what is kept
        m = min(32, n - i)
        b = torch.cat([_matrix(m, 2 * I, H, dtype, g), _matrix(m, H, I, dtype, g)], 1)
        if out is None:
            out = torch.empty((n, b.shape[1]), dtype=torch.uint8, device="cuda")
        out[i:i + m] = b
    return out


def _dense(blob, H, I, dtype):
    """(W_gu [2I x H], W_d [H x I]) of one blob in 64 bits."""
    res, off = [], 0
    for rows, cols in ((2 * I, H), (H, I)):
        if dtype == "int4":
            nq = rows * cols // 2
            b = blob[off:off + nq]
            q = torch.stack([b & 15, b >> 4], 1).to(torch.float64)
            q = torch.where(q > 7, q - 16, q).view(rows, cols // 128, 128)
            ns = rows * (cols // 128) * 2
            s = blob[off + nq:off + nq + ns].clone().view(torch.bfloat16).to(torch.float64).view(rows, cols // 128, 1)
            res.append((q * s).view(rows, cols))
            off += nq + ns
        else:
            t = torch.float32 if dtype == "f32" else torch.bfloat16
            n = rows * cols * (4 if dtype == "f32" else 2)
            res.append(blob[off:off + n].clone().view(t).to(torch.float64).view(rows, cols))
            off += n
    return res


def _zipf_ids(T, E, k, g, overlap=0.0):
    """T tokens' expert sets: popularity rank^-1.1 over a random order of the experts, drawn without
    replacement; each expert of the token before is kept with probability `overlap`."""
    logp = -1.1 * torch.log(torch.arange(1, E + 1, device="cuda", dtype=torch.float32))
    logp = logp[torch.randperm(E, generator=g, device="cuda")]
    u = torch.rand((T, E), generator=g, device="cuda").clamp_(1e-12, 1 - 1e-7)
    score = logp - torch.log(-torch.log(u))
    if overlap:
        keep = torch.rand((T, E), generator=g, device="cuda") < overlap
        prev = None
        for t in range(T):
            if prev is not None:
                score[t] += 100.0 * (prev & keep[t]) - 100.0 * (prev & ~keep[t])
            prev = torch.zeros(E, dtype=torch.bool, device="cuda")
            prev[score[t].topk(k).indices] = True
    return score.topk(k, dim=1).indices.to(torch.int32)


def _inputs(case, seed):
    """Every tensor of a case, made from the seed alone."""
    g = _gen(seed)
    c, kind = case, case["kind"]
    if kind == "route":
        t = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
        return {"x": _normal((c["T"], c["H"]), g), "w": _normal((c["E"], c["H"]), g, SIGMA).to(t)}
    if kind in ("ffn", "prefill"):
        T, H, I, E, k = c["T"], c["H"], c["I"], c["E"], c["k"]
        r = {"x": _normal((T, H), g)}
        if kind == "ffn" or c["zipf"]:
            r["ids"] = _zipf_ids(T, E, k, g)
        else:
            r["ids"] = torch.rand((T, E), generator=g, device="cuda").topk(k, dim=1).indices.to(torch.int32)
        r["weights"] = torch.softmax(_normal((T, k), g), 1).sort(1, descending=True).values.contiguous()
        r["slot_of"] = torch.randperm(E, generator=g, device="cuda").to(torch.int32)  # as a cache leaves them
        r["pool"] = _experts(E, H, I, c["dtype"], g)
        r["shared"] = _experts(1, H, I, c["dtype"], g)[0] if c["shared"] else None
        return r
    if kind == "attention":
        H, nh, kv, d, mp = c["H"], c["heads"], c["kv"], c["d"], c["max_pos"]
        b = torch.bfloat16
        return {"x": _normal((H,), g), "w_qkv": _normal(((nh + 2 * kv) * d, H), g, SIGMA).to(b),
                "w_o": _normal((H, nh * d), g, SIGMA).to(b),
                "k_cache": _normal((kv, d // 8, mp, 8), g).to(b), "v_cache": _normal((kv, mp, d), g).to(b)}
    L, H, I, E, k, n = c["L"], c["H"], c["I"], c["E"], c["k"], c["tokens"]
    r = {"x": _normal((n, 1, H), g), "router": [_normal((E, H), g, SIGMA).to(torch.bfloat16) for _ in range(L)]}
    bias = torch.zeros((n, L, 1, E), device="cuda")
    for l in range(L):
        bias[:, l, 0].scatter_(1, _zipf_ids(n, E, k, g, overlap=0.7).long(), MASK)
    r["bias"] = bias
    # under a budget the layers share one host copy of the experts (their cache entries stay apart)
    r["experts"] = _experts(E if c["slots"] else L * E, H, I, c["dtype"], g)
    r["shared"] = [_experts(1, H, I, c["dtype"], g)[0] for _ in range(L)] if c["shared"] else None
    return r


def prepare(case, seed):
    moe.moe_init(torch.cuda.current_device())
    s = _inputs(case, seed)
    c, kind = case, case["kind"]
    s["case"] = c
    if kind == "route":
        T, E, k = c["T"], c["E"], c["k"]
        s["logits"] = torch.empty((T, E), device="cuda")
        s["ids"] = torch.empty((T, k), dtype=torch.int32, device="cuda")
        s["weights"] = torch.empty((T, k), device="cuda")
        s["x_norm"] = torch.empty((T, c["H"]), device="cuda")
    elif kind in ("ffn", "prefill"):
        s["eb"] = s["pool"].shape[1]
        s["y"] = torch.empty((c["T"], c["H"]), device="cuda")
        n = (moe.moe_ffn_workspace_bytes(c["T"], c["k"], c["I"]) if kind == "ffn" else
             moe.moe_prefill_workspace_bytes(c["T"], c["k"], c["E"], c["H"], c["I"]))
        s["ws"] = torch.empty(max(n, 256), dtype=torch.uint8, device="cuda")
        # slot s holds the expert whose slot_of is s
        order = torch.empty_like(s["slot_of"])
        order[s["slot_of"].long()] = torch.arange(c["E"], device="cuda", dtype=torch.int32)
        s["pool"] = s["pool"][order.long()].contiguous()
    elif kind == "attention":
        n = moe.moe_attention_workspace_bytes(c["heads"], c["kv"], c["d"], c["max_pos"])
        s["ws"] = torch.empty(max(n, 256), dtype=torch.uint8, device="cuda")
    else:
        L, E, n = c["L"], c["E"], c["tokens"]
        ex = s.pop("experts")
        eb = ex.shape[1]
        host = moe.PinnedBuffer(ex.numel())
        torch.from_numpy(host.array).copy_(ex.view(-1))
        del ex
        shared_bytes = L * eb if c["shared"] else 0
        slots = c["slots"] or L * E
        cache = moe.ExpertCache(L, E, eb, slots * eb + shared_bytes, host.ptr, 0 if c["slots"] else E * eb, eb,
                                reserved_bytes=shared_bytes, preload=not c["slots"], device=bool(c["slots"]))
        cache.host_store = host  # lives as long as the cache
        s["stack"] = moe.MoeStack(cache, c["H"], c["I"], E, c["k"], DT[c["dtype"]], moe.MOE_BF16, s["router"],
                                  s["shared"])
        s["xs"] = torch.empty_like(s["x"])
        s["logits"] = torch.empty((n, L, 1, E), device="cuda")
        s["step"] = 0
    torch.cuda.synchronize()
    return s


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "route":
        moe.moe_route_topk(s["x"], s["w"], DT[c["dtype"]], c["k"], logits=s["logits"], ids=s["ids"],
                           weights=s["weights"], rmsnorm=True, x_norm=s["x_norm"])
        return s["logits"], s["ids"], s["weights"], s["x_norm"]
    if kind == "ffn":
        a = (s["x"], s["ids"], s["weights"], s["pool"], s["eb"], DT[c["dtype"]], c["I"], c["E"])
        kw = dict(slot_of=s["slot_of"], shared_w=s["shared"], y_out=s["y"])
        if c["noalloc"]:
            return moe.moe_expert_ffn_grouped_noalloc(*a, **kw)
        return moe.moe_expert_ffn_grouped(*a, workspace=s["ws"], **kw)
    if kind == "prefill":
        return moe.moe_prefill_grouped(s["x"], s["ids"], s["weights"], s["pool"], s["eb"], DT[c["dtype"]], c["I"],
                                       c["E"], slot_of=s["slot_of"], shared_w=s["shared"], y_out=s["y"],
                                       workspace=s["ws"])
    if kind == "attention":
        x = s["x"].clone()
        moe.moe_attention_decode(x, s["w_qkv"], s["w_o"], s["k_cache"], s["v_cache"], c["p"], c["heads"], c["kv"],
                                 workspace=s["ws"])
        return x, s["k_cache"], s["v_cache"]
    s["xs"].copy_(s["x"])
    for t in range(c["tokens"]):
        s["stack"].decode_step(s["step"], s["xs"][t], s["bias"][t], logits_out=s["logits"][t])
        s["step"] += 1
    return s["xs"], s["logits"]


# -------------------------------------------------------------------------------------------------- work ---
def _expert_bytes(H, I, dtype):
    n = 3 * H * I
    return n // 2 + n // 64 if dtype == "int4" else n * (4 if dtype == "f32" else 2)


def _distinct(T, E, k, zipf):
    """Distinct experts that T tokens choose, on average."""
    rng = np.random.default_rng(0)
    logp = -1.1 * np.log(np.arange(1, E + 1)) if zipf else np.zeros(E)
    n = [np.unique(np.argpartition(-(logp + rng.gumbel(size=(T, E))), k - 1, axis=1)[:, :k]).size for _ in range(8)]
    return float(np.mean(n))


def work(case):
    c, kind = case, case["kind"]
    H = c["H"]
    if kind == "route":
        T, E, k = c["T"], c["E"], c["k"]
        b = T * H * 4 * 2 + E * H * (4 if c["dtype"] == "f32" else 2) + T * E * 4 + T * k * 8
        return {"bytes": b, "flops": 2 * T * E * H}
    if kind in ("ffn", "prefill"):
        T, I, E, k = c["T"], c["I"], c["E"], c["k"]
        n = _distinct(T, E, k, kind == "ffn" or c["zipf"]) + (1 if c["shared"] else 0)
        rows = T * k + (T if c["shared"] else 0)
        return {"bytes": int(n * _expert_bytes(H, I, c["dtype"])) + T * H * 8 + T * k * 8,
                "flops": 2 * rows * 3 * H * I}
    if kind == "attention":
        nh, kv, d, n = c["heads"], c["kv"], c["d"], c["p"] + 1
        w = (nh + 2 * kv) * d * H + H * nh * d
        return {"bytes": 2 * w + 4 * kv * n * d + 8 * H, "flops": 2 * w + 4 * nh * d * n}
    L, I, E, k = c["L"], c["I"], c["E"], c["k"]
    ne = k + (1 if c["shared"] else 0)
    layer = ne * _expert_bytes(H, I, c["dtype"]) + E * H * 2
    return {"bytes": c["tokens"] * (L * (layer + E * 8) + 8 * H),
            "flops": c["tokens"] * L * (2 * ne * 3 * H * I + 2 * E * H)}


def tolerance(case):
    c, kind = case, case["kind"]
    if kind == "route":  # 32-bit sums; "differ": tokens whose ranked logits tie to the last bits
        return {"rel": 1e-6, "max": 4e-5, "differ": 0.002}
    if kind == "ffn":
        # one int4 token: activations in fp16; otherwise 32-bit sums over exact weights
        return {"rel": 1.5e-3} if c["dtype"] == "int4" else {"rel": 1.5e-6}
    if kind == "prefill":  # x and the SwiGLU activations in bf16 on the matrix cores
        return {"rel": 1.2e-2, "max": 0.2}
    if kind == "attention":  # "max": a new key or value at a bf16 rounding boundary
        return {"rel": 1e-5, "max": 4e-2}
    return {"rel": 1e-3} if c["dtype"] == "int4" else {"rel": 3e-6}


# ------------------------------------------------------------------------------------------------- exact ---
def _norm(x):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS)


def _ffn(x, gu, d):
    a = x @ gu.T
    g, u = a[:, 0::2], a[:, 1::2]
    return (g / (1 + torch.exp(-g)) * u) @ d.T


def _moe(x, ids, w, experts, shared, H, I, dtype):
    """sum_j w_j FFN_{ids_j}(x) (+ shared), expert e's blob at experts[e]."""
    y = torch.zeros_like(x)
    for e in torch.unique(ids).tolist():
        t, j = torch.nonzero(ids == e, as_tuple=True)
        y.index_add_(0, t, _ffn(x[t], *_dense(experts[e], H, I, dtype)) * w[t, j].unsqueeze(1))
    if shared is not None:
        y += _ffn(x, *_dense(shared, H, I, dtype))
    return y


def _rope(v, p, theta):
    d = v.shape[-1]
    i = torch.arange(d // 2, device=v.device, dtype=torch.float64)
    ang = p * theta ** (-2 * i / d)
    a, b = v[..., :d // 2], v[..., d // 2:]
    return torch.cat([a * torch.cos(ang) - b * torch.sin(ang), b * torch.cos(ang) + a * torch.sin(ang)], -1)


def exact(case, seed):
    c, kind = case, case["kind"]
    s = _inputs(case, seed)
    f8 = torch.float64
    if kind == "route":
        h = _norm(s["x"].to(f8))
        z = h @ s["w"].to(f8).T
        top = z.topk(c["k"], dim=1)
        return z, top.indices.to(torch.int32), torch.softmax(top.values, 1), h
    if kind in ("ffn", "prefill"):
        return _moe(s["x"].to(f8), s["ids"], s["weights"].to(f8), s["pool"], s["shared"], c["H"], c["I"], c["dtype"])
    if kind == "attention":
        nh, kv, d, p = c["heads"], c["kv"], c["d"], c["p"]
        x = s["x"].to(f8)
        qkv = s["w_qkv"].to(f8) @ _norm(x)
        q = _rope(_norm(qkv[:nh * d].view(nh, d)), p, 1.0e6)
        kn = _rope(_norm(qkv[nh * d:(nh + kv) * d].view(kv, d)), p, 1.0e6)
        kc, vc = s["k_cache"].clone(), s["v_cache"].clone()
        kc[:, :, p] = kn.view(kv, d // 8, 8).to(torch.bfloat16)
        vc[:, p] = qkv[(nh + kv) * d:].view(kv, d).to(torch.bfloat16)
        K = kc.permute(0, 2, 1, 3).reshape(kv, -1, d)[:, :p + 1].to(f8).repeat_interleave(nh // kv, 0)
        V = vc[:, :p + 1].to(f8).repeat_interleave(nh // kv, 0)
        prob = torch.softmax((K * q.unsqueeze(1)).sum(-1) / math.sqrt(d), 1)
        att = (prob.unsqueeze(-1) * V).sum(1).reshape(-1)
        return x + s["w_o"].to(f8) @ att, kc.to(f8), vc.to(f8)
    L, H, I, E, k, n = c["L"], c["H"], c["I"], c["E"], c["k"], c["tokens"]
    x = s["x"].to(f8).view(n, H)
    logits = torch.empty((n, L, 1, E), dtype=f8, device="cuda")
    for l in range(L):
        h = _norm(x)
        z = h @ s["router"][l].to(f8).T + s["bias"][:, l, 0].to(f8)
        logits[:, l, 0] = z
        top = z.topk(k, dim=1)
        first = 0 if c["slots"] else l * E
        x = x + _moe(h, top.indices, torch.softmax(top.values, 1), s["experts"][first:first + E],
                     s["shared"][l] if c["shared"] else None, H, I, c["dtype"])
    return x.view(n, 1, H), logits
