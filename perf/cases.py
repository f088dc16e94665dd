"""The workloads whose time on one MI355X this repository answers for.

A case is a dict of plain values:
  kind         "decode"     one token per sequence against block caches of one length
               "generate"   the step of a serving loop: append one token per sequence, decode at ragged lengths
               "forward"    prefill: representatives, selection, sparse attention (Lq < Lk: a later chunk of a prompt)
               "train"      the same with the backward, workspace kept and index reused (an engine's own step)
               "autograd"   the same through torch's autograd
  batch, lq, lk, hq, hkv, d       sizes (B, query rows, keys or cache capacity, query and KV heads, head dim)
  m, top_k, n_init, window        Algorithm 1: block size, free picks, init blocks, local window in tokens
  dtype        "bf16" or "fp32"
  softmax_sum  blocks ranked by the heads' summed softmax instead of their summed logits

Inputs follow paper_2601_02819_amd.inputs: standard normals and a Bernoulli(0.08)
punctuation mask, drawn here on the GPU.  Heads 16/8 of dim 128 and the 32k
lengths are the paper's Qwen3-0.6B-like training model.
"""
import math
import random

import torch

from paper_2601_02819_amd import phsa


def _case(kind, batch, lq, lk, hq=16, hkv=8, d=128, m=64, top_k=12, n_init=1, window=0, dtype="bf16",
          softmax_sum=False):
    return {"kind": kind, "batch": batch, "lq": lq, "lk": lk, "hq": hq, "hkv": hkv, "d": d, "m": m, "top_k": top_k,
            "n_init": n_init, "window": window, "dtype": dtype, "softmax_sum": softmax_sum}


PAPER = dict(m=16, top_k=16, n_init=8, window=512)  # the paper's 32k geometry: 57 blocks of 16 tokens


def listed():
    return [
        # one user's chat: a single sequence, one token, latency is everything
        dict(_case("decode", 1, 1, 8192, top_k=14), name="decode_1x8k"),
        # a few long-context users in the paper's geometry (T = 2048 representatives each)
        dict(_case("decode", 6, 1, 32768, **PAPER), name="decode_6x32k_paper"),
        # a full serving batch on 32k caches (the benchmark's decode step)
        dict(_case("decode", 64, 1, 32768), name="decode_64x32k"),
        # continuous batching: ragged lengths, an odd number of sequences, cache kept up to date
        dict(_case("generate", 23, 1, 16384), name="generate_23_ragged"),
        # a short prompt's prefill: a chain of small launches
        dict(_case("forward", 1, 1024, 1024, top_k=6), name="prefill_1k"),
        # the 8k prefill
        dict(_case("forward", 1, 8192, 8192, top_k=14), name="prefill_8k"),
        # chunked prefill: an odd number of new rows at the end of a 20k prompt
        dict(_case("forward", 1, 1000, 20480), name="prefill_chunk_1000_of_20k"),
        # the 16k prefill with blocks ranked by summed softmax (Eq. 8 read per head)
        dict(_case("forward", 1, 16384, 16384, softmax_sum=True), name="prefill_16k_softmax_sum"),
        # fine-tuning on short sequences: head dim 64, four query heads per KV head, a ragged length
        dict(_case("autograd", 6, 2112, 2112, hq=16, hkv=4, d=64, top_k=8), name="train_6x2112_g4_d64"),
        # float32 training on a small model (checks, ablations): the tiny_fp32 workload
        dict(_case("autograd", 1, 1024, 1024, hq=2, hkv=1, d=64, top_k=2, dtype="fp32"), name="train_1k_fp32"),
        # the benchmark's training step
        dict(_case("train", 4, 32768, 32768), name="train_4x32k"),
        # the same tokens in the paper's geometry
        dict(_case("train", 4, 32768, 32768, **PAPER), name="train_4x32k_paper"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(["decode", "generate", "forward", "forward", "train", "autograd", "autograd"])
    fp32 = kind == "autograd" and rng.random() < 0.4
    if fp32:  # small problems: float32 runs on the vector units
        hkv, group, d = rng.choice([1, 2, 4]), rng.choice([1, 2, 4]), rng.choice([64, 64, 128])
        m = rng.choice([16, 32, 64, 64])
        lk = m * max(1, _log(rng, 256, 4096) // m)
        return _case(kind, rng.randint(1, 2), lk, lk, hq=hkv * group, hkv=hkv, d=d, m=m, top_k=rng.randint(2, 12),
                     n_init=rng.randint(1, 2), window=m * rng.choice([0, 0, 2, 4]), dtype="fp32")
    hkv, group = rng.choice([(8, 2), (8, 2), (8, 1), (4, 4), (2, 8)])
    geo = rng.choice([dict(m=64, top_k=rng.randint(4, 16)), dict(m=64, top_k=12),
                      dict(m=64, top_k=rng.randint(4, 12), window=rng.choice([64, 256, 512])),
                      dict(m=32, top_k=rng.randint(4, 16), n_init=4, window=256), PAPER])
    d = rng.choice([64, 128, 128])
    most = 32768 if geo["m"] == 16 else 65536  # at most 2048 blocks
    tokens = 0.8 * 4 * 32768 * 8 / hkv          # query rows of all sequences: below the largest listed case
    if kind in ("decode", "generate"):
        lk = 64 * (_log(rng, 1024, most) // 64)
        batch = max(1, min(_log(rng, 1, 96), int(64 * 32768 / lk)))
        return _case(kind, batch, 1, lk, hq=hkv * group, hkv=hkv, d=d, softmax_sum=rng.random() < 0.2, **geo)
    lk = 64 * (_log(rng, 512, 32768) // 64)
    lq = lk
    if kind == "forward" and rng.random() < 0.4:
        lq = min(lk, _log(rng, 64, 8192))
    batch = max(1, min(_log(rng, 1, 12), int(tokens * 2 / group / lk)))
    soft = kind == "forward" and rng.random() < 0.25
    return _case(kind, batch, lq, lk, hq=hkv * group, hkv=hkv, d=d, softmax_sum=soft, **geo)


def _cfg(c):
    return phsa.Config(block_size=c["m"], top_k=c["top_k"], n_init_blocks=c["n_init"], window=c["window"],
                       softmax_sum=c["softmax_sum"])


def _inputs(c, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    B, Lq, Lk, d = c["batch"], c["lq"], c["lk"], c["d"]

    def normal(*shape):
        return torch.randn(*shape, generator=gen, device="cuda").to(dt)

    x = {"q": normal(B, Lq, c["hq"], d), "k": normal(B, Lk, c["hkv"], d), "v": normal(B, Lk, c["hkv"], d)}
    if c["kind"] in ("train", "autograd"):
        x["do"] = normal(B, Lq, c["hq"], d)
    x["punct"] = (torch.rand(B, Lk, generator=gen, device="cuda") < 0.08).to(torch.uint8)
    if c["kind"] == "generate":
        x["k_new"], x["v_new"] = normal(B, c["hkv"], d), normal(B, c["hkv"], d)
        x["punct_new"] = (torch.rand(B, generator=gen, device="cuda") < 0.08).to(torch.uint8)
        # lengths before the step: anywhere in the upper three quarters of the cache, room for one token;
        # every fourth sequence completes a block with this token
        n = torch.randint(Lk // 4, Lk, (B,), generator=gen, device="cuda", dtype=torch.int32)
        n[::4] = (n[::4] // c["m"] + 1) * c["m"] - 1
        x["lens"] = n
    return x


def prepare(c, seed):
    x, cfg = _inputs(c, seed), _cfg(c)
    s = {"case": c, "cfg": cfg, **x}
    if c["kind"] in ("decode", "generate"):
        s["kc"] = phsa.compress(x["k"], x["punct"], cfg)  # the cache's representatives, kept by the serving program
        if c["kind"] == "generate":
            s["clen"] = x["lens"].clone()
    elif c["kind"] in ("forward", "train"):
        p = phsa.make_params(cfg, c["batch"], c["lq"], c["lk"], c["hq"], c["hkv"], c["d"], x["q"].dtype)
        need = phsa.workspace_size(p, phsa.OP_FORWARD)
        if c["kind"] == "train":
            need = max(need, phsa.workspace_size(p, phsa.OP_ATTN_BWD))
        s["ws"] = torch.empty(need, dtype=torch.uint8, device="cuda") if need else None
    else:
        for n in "qkv":
            s[n].requires_grad_(True)
    return s


def run(s):
    kind, cfg = s["case"]["kind"], s["cfg"]
    if kind == "decode":
        sel, o, lse = phsa.decode(s["q"], s["k"], s["v"], s["kc"], cfg)
        return {"sel": sel, "o": o, "lse": lse}
    if kind == "generate":
        s["clen"].copy_(s["lens"])  # the scheduler owns the lengths
        phsa.cache_append(s["k_new"], s["v_new"], s["punct_new"], s["k"], s["v"], s["punct"], s["clen"], s["kc"], cfg)
        sel, o, lse = phsa.decode_varlen(s["q"], s["k"], s["v"], s["kc"], s["clen"], cfg)
        return {"sel": sel, "o": o, "lse": lse, "clen": s["clen"], "kc": s["kc"]}
    if kind == "forward":
        kc, sel, o, lse = phsa.forward(s["q"], s["k"], s["v"], s["punct"], cfg, s["ws"])
        return {"kc": kc, "sel": sel, "o": o, "lse": lse}
    if kind == "train":
        kc, sel, o, lse = phsa.forward(s["q"], s["k"], s["v"], s["punct"], cfg, s["ws"])
        dq, dk, dv = phsa.attn_bwd(s["q"], s["k"], s["v"], o, s["do"], lse, sel, cfg, s["ws"], reuse_index=True)
        return {"sel": sel, "o": o, "dq": dq, "dk": dk, "dv": dv}
    with torch.no_grad():
        sel = phsa.select(s["q"], phsa.compress(s["k"], s["punct"], cfg), s["case"]["lk"], cfg)
    o = phsa.SparseAttention.apply(s["q"], s["k"], s["v"], sel, cfg)
    dq, dk, dv = torch.autograd.grad(o, (s["q"], s["k"], s["v"]), s["do"])
    return {"sel": sel, "o": o.detach(), "dq": dq, "dk": dk, "dv": dv}


def work(c):
    B, Lq, Lk, Hq, Hkv, d, m = (c[x] for x in ("batch", "lq", "lk", "hq", "hkv", "d", "m"))
    es = 2 if c["dtype"] == "bf16" else 4
    ksel = c["n_init"] + c["window"] // m + 1 + c["top_k"]
    scored = keys = 0  # blocks scored and keys attended, over the query rows of one (sequence, KV head)
    for cur in range((Lk - Lq) // m, (Lk - 1) // m + 1):
        rows = min(Lk, (cur + 1) * m) - max(Lk - Lq, cur * m)
        lo = max(0, cur - c["window"] // m)
        if c["top_k"]:
            scored += rows * (cur if c["softmax_sum"] else max(0, lo - c["n_init"]))
        keys += rows * (min(cur + 1, ksel) * m - (m - 1) / 2 * (Lq > 1))
    score = 2 * d * scored * B * Hkv * (Hq // Hkv if c["softmax_sum"] else 1)
    attend = 4 * d * keys * B * Hq
    kc, sel, lse = B * Hkv * (Lk // m) * d * 4, B * Hkv * Lq * ksel * 4, B * Hq * Lq * 4
    q, kv = B * Lq * Hq * d * es, B * Lk * Hkv * d * es
    if c["kind"] in ("decode", "generate"):
        if c["kind"] == "generate":  # lengths lie evenly in the upper three quarters
            kc, score = kc * 5 // 8, score * 5 // 8
        nbytes = kc + 2 * B * Hkv * min(ksel, Lk // m) * m * d * es + 2 * q + sel + lse
        if c["kind"] == "generate":  # the token's row in and out, a quarter of the sequences pool a block
            nbytes += 4 * B * Hkv * d * es + B * Hkv * m * d * es // 4
        return {"bytes": nbytes, "flops": score + attend}
    if c["kind"] == "forward":
        return {"bytes": 2 * q + 2 * kv + B * Lk + kc + sel + lse, "flops": score + attend}
    # backward: Q, K, V, dO in, O, dQ, dK, dV and sel out
    return {"bytes": 4 * q + 4 * kv + B * Lk + sel, "flops": score + 3.5 * attend}


def tolerance(c):
    # float32 sums in another order; bf16 results and partials rounded at other
    # places (measured against float64: decode 0.0017, prefill and training 0.0025
    # to 0.0053, float32 8e-7).  Blocks whose scores tie within the float32
    # rounding of a dot product may swap: that moves a few entries of a row's sel
    # and a few tenths of the row's own output.
    if c["dtype"] == "fp32":
        return {"rel": 1e-5, "max": 1e-3, "differ": 1e-3}
    if c["kind"] in ("decode", "generate"):
        return {"rel": 8e-3, "max": 0.3, "differ": 1e-3}
    return {"rel": 2e-2, "max": 1.0, "differ": 1e-3}


def _representatives(c, k, punct):
    """Eq. 6-8 in float64: [B, Hkv, T, d]."""
    B, Lk, H, d = k.shape
    kb = k.double().view(B, Lk // c["m"], c["m"], H, d)
    pb = punct.double().view(B, Lk // c["m"], c["m"], 1, 1)
    n = pb.sum(2)
    m0 = kb.mean(2)
    mp = (kb * pb).sum(2) / n.clamp_min(1)
    return torch.where(n > 0, 0.5 * m0 + 0.5 * mp, m0).permute(0, 2, 1, 3)


def _select(c, q, kc, pos):
    """Blocks kept by rows at positions pos [n]: q [n, G, d], kc [T, d] of one KV head -> bool [n, T]."""
    T, m, k = kc.shape[0], c["m"], c["top_k"]
    t = torch.arange(T, device=q.device)[None]
    cur = (pos // m)[:, None]
    lo = (cur - c["window"] // m).clamp_min(0)
    x = (q.reshape(-1, q.shape[-1]) @ kc.T).view(q.shape[0], q.shape[1], T) / math.sqrt(c["d"])
    if c["softmax_sum"]:
        x = x.masked_fill((t >= cur)[:, None], -math.inf)
        x = torch.logsumexp(x - torch.logsumexp(x, 2, keepdim=True), 1)
    else:
        x = x.sum(1)
    kept = ((t < c["n_init"]) | (t >= lo)) & (t <= cur)
    cand = (t >= c["n_init"]) & (t < lo)
    if k:
        best, at = x.masked_fill(~cand, -math.inf).nan_to_num(nan=-math.inf).topk(min(k, T), 1)
        kept = kept | (torch.zeros_like(kept).scatter(1, at, best > -math.inf) & cand)
    return kept


def _sel_rows(c, kept):
    ksel = c["n_init"] + c["window"] // c["m"] + 1 + c["top_k"]
    T = kept.shape[1]
    ids = torch.where(kept, torch.arange(T, device=kept.device)[None], T).sort(1).values[:, :ksel]
    ids = torch.nn.functional.pad(ids, (0, ksel - ids.shape[1]), value=T)
    return torch.where(ids < T, ids, -1).to(torch.int32)


def exact(c, seed):
    x = _inputs(c, seed)
    B, Lq, Lk, Hq, Hkv, d, m = (c[n] for n in ("batch", "lq", "lk", "hq", "hkv", "d", "m"))
    G, scale = Hq // Hkv, 1 / math.sqrt(c["d"])
    back = c["kind"] in ("train", "autograd")
    if c["kind"] == "generate":
        at = x["lens"].long()
        rows = torch.arange(B, device="cuda")
        x["k"][rows, at], x["v"][rows, at], x["punct"][rows, at] = x["k_new"], x["v_new"], x["punct_new"]
    kc = _representatives(c, x["k"], x["punct"])
    sel = torch.empty(B, Hkv, Lq, c["n_init"] + c["window"] // m + 1 + c["top_k"], dtype=torch.int32, device="cuda")
    o = torch.empty(B, Lq, Hq, d, dtype=torch.float64, device="cuda")
    lse = torch.empty(B, Hq, Lq, dtype=torch.float64, device="cuda")
    if back:
        dq, dk, dv = torch.empty_like(o), *(torch.zeros(B, Lk, Hkv, d, dtype=torch.float64, device="cuda") for _ in "kv")
    step = 2048
    for b in range(B):
        for g in range(Hkv):
            k, v = x["k"][b, :, g].double(), x["v"][b, :, g].double()
            for i in range(0, Lq, step):
                n = min(step, Lq - i)
                q = x["q"][b, i:i + n, g * G:(g + 1) * G].double()
                pos = torch.arange(Lk - Lq + i, Lk - Lq + i + n, device="cuda")
                if c["kind"] == "generate":
                    pos = x["lens"][b:b + 1].long()
                kept = _select(c, q, kc[b, g], pos)
                sel[b, g, i:i + n] = _sel_rows(c, kept)
                end = Lk if c["kind"] == "generate" else Lk - Lq + i + n
                ok = kept.repeat_interleave(m, 1)[:, :end] & (torch.arange(end, device="cuda")[None] <= pos[:, None])
                for h in range(G):
                    s = (q[:, h] @ k[:end].T).mul_(scale).masked_fill_(~ok, -math.inf)
                    l = torch.logsumexp(s, 1)
                    p = s.sub_(l[:, None]).exp_()
                    oh = p @ v[:end]
                    o[b, i:i + n, g * G + h], lse[b, g * G + h, i:i + n] = oh, l
                    if back:
                        do = x["do"][b, i:i + n, g * G + h].double()
                        dv[b, :end, g] += p.T @ do
                        ds = p.mul_((do @ v[:end].T).sub_((do * oh).sum(1, keepdim=True)))
                        dq[b, i:i + n, g * G + h] = ds @ k[:end] * scale
                        dk[b, :end, g] += ds.T @ q[:, h] * scale
    if back:
        return {"sel": sel, "o": o, "dq": dq, "dk": dk, "dv": dv}
    if c["kind"] == "decode":
        return {"sel": sel, "o": o, "lse": lse}
    if c["kind"] == "forward":
        return {"kc": kc, "sel": sel, "o": o, "lse": lse}
    # the blocks past a sequence's length hold what compress made of the unwritten cache; they never change
    return {"sel": sel, "o": o, "lse": lse, "clen": x["lens"] + 1, "kc": None}
