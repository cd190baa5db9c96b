"""The calls whose speed matters to a user of this library, as cases to time.

Each case is one call (or one forward + backward) of an attention layer through
`paper_2502_13189_amd.binding`, with everything such a program has in hand
before the call already on the GPU and cu_seqlens on the host:

  prefill       moba_forward over a packed batch of sequences
  train         moba_forward, then moba_backward with its out and lse
  decode        moba_decode, one new query per sequence, the loop's block means kept
  decode_fresh  moba_decode that computes the block means itself
  full_prefill, full_train, full_decode
                the same with full causal attention (a model's full-attention
                layers, and the generation phase of a MoBA model)

Inputs are Gaussian with a per-block key offset, as in the repository's own
workloads; `packed` cases pass q, k and v as views of one fused projection.
"""
import math

import torch

from paper_2502_13189_amd import binding

DEV = "cuda:0"
D = 128
SCALE = 1.0 / math.sqrt(D)


def _case(name, kind, seqlens, hq, hkv, block=0, topk=0, dtype="bf16", packed=False):
    return {"name": name, "kind": kind, "seqlens": ",".join(str(x) for x in seqlens), "hq": hq,
            "hkv": hkv, "block": block, "topk": topk, "dtype": dtype, "packed": packed}


def listed():
    return [
        # the 1K fp32 workload: one short sequence, one head (checks, tiny models)
        _case("prefill_f32_1k", "prefill", (1024,), 1, 1, 128, 3, "f32"),
        # fp32 of a layer's size, ragged, GQA (reference runs and fp32 training)
        _case("prefill_f32_ragged", "prefill", (4096, 1500, 777), 8, 2, 256, 4, "f32"),
        # the smallest bf16 calls: two short ragged prompts
        _case("prefill_small", "prefill", (700, 333), 8, 2, 128, 3),
        # the 8K scaling-law setting, MHA
        _case("prefill_8k", "prefill", (8192,), 32, 32, 512, 3),
        # many small blocks: the finest point of the granularity sweep
        _case("prefill_32k_fine", "prefill", (32768,), 32, 8, 256, 32),
        # a packed batch of ragged sequences, q/k/v from one projection
        _case("prefill_varlen", "prefill", (4096, 12288, 30000, 65536), 32, 32, 1024, 4,
              packed=True),
        # the largest call: the 1M-token prefill of the long-context model
        _case("prefill_1m", "prefill", (1048576,), 32, 8, 4096, 12),
        # a full-attention layer of the hybrid model
        _case("full_prefill_16k", "full_prefill", (16384,), 32, 8),
        # one training pass of a layer: a short ragged batch, and the 32K hybrid setting
        _case("train_small", "train", (1000, 1, 517), 8, 2, 128, 3),
        _case("train_32k", "train", (32768,), 32, 8, 2048, 3),
        # generation: MoBA against the 1M-token cache; full attention for a ragged batch
        _case("decode_1m", "decode", (1048576,), 32, 8, 4096, 12),
        _case("full_decode_batch", "full_decode",
              (30011, 512, 9000, 65536, 1, 4097, 16384, 2300), 32, 8),
    ]


#: kind, dtype, share of the draws, tokens from, tokens to
_KINDS = [
    ("prefill", "bf16", 4, 256, 131072),
    ("prefill", "f32", 2, 256, 8192),
    ("full_prefill", "bf16", 1, 256, 24576),
    ("full_prefill", "f32", 1, 256, 4096),
    ("train", "bf16", 3, 256, 49152),
    ("full_train", "bf16", 1, 256, 16384),
    ("decode", "bf16", 2, 256, 1 << 20),
    ("decode_fresh", "bf16", 1, 256, 1 << 19),
    ("full_decode", "bf16", 1, 256, 1 << 20),
]
#: query heads, kv-heads
_HEADS = [(1, 1), (4, 4), (8, 2), (12, 4), (16, 2), (32, 8), (32, 32)]


def draw(rng):
    while True:
        kind, dtype, _, lo, hi = rng.choices(_KINDS, [x[2] for x in _KINDS])[0]
        T = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
        n = rng.choice((1, 1, 2, 3, 5, 8))
        cuts = sorted({0, T} | {rng.randrange(1, T) for _ in range(n - 1)})
        lens = [b - a for a, b in zip(cuts, cuts[1:])]
        hq, hkv = rng.choice(_HEADS)
        # block sizes of a MoBA model, odd ones among them; at least four blocks in the batch
        B = int(round(math.exp(rng.uniform(math.log(64), math.log(max(65, min(4096, T // 4)))))))
        if rng.random() < 0.6:
            B = 1 << (B.bit_length() - 1)
        topk = rng.choice((2, 3, 3, 4, 4, 6, 8, 12, 16, 24, 32))
        if kind.startswith("full"):
            B = topk = 0
        c = _case("", kind, lens, hq, hkv, B, topk, dtype,
                  packed="decode" not in kind and rng.random() < 0.25)
        del c["name"]
        if work(c)["flops"] < (1e11 if dtype == "f32" else 2e13):
            return c


# ------------------------------------------------------------------- inputs
def _lens(case):
    return [int(x) for x in case["seqlens"].split(",")]


def _inputs(case, seed):
    """q, k, v (and dout) of a case, from the seed alone."""
    lens = _lens(case)
    T, hq, hkv = sum(lens), case["hq"], case["hkv"]
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    gen = torch.Generator(device=DEV).manual_seed(seed)
    decode = "decode" in case["kind"]

    def randn(shape, dtype=torch.float32):
        return torch.randn(shape, generator=gen, device=DEV, dtype=torch.float32).to(dtype)

    # one offset vector per block of keys and kv-head: what the gate looks for
    B = case["block"] or 2048
    ids, nb = [], 0
    for L in lens:
        ids.append(torch.arange(L, device=DEV) // B + nb)
        nb += -(-L // B)
    ids = torch.cat(ids)
    off = randn((nb, hkv, D)) * 0.5
    if case["packed"]:
        qkv = torch.empty((T, hq + 2 * hkv, D), device=DEV, dtype=dt)
        q, k, v = qkv[:, :hq], qkv[:, hq:hq + hkv], qkv[:, hq + hkv:]
    else:
        q = torch.empty((len(lens) if decode else T, hq, D), device=DEV, dtype=dt)
        k = torch.empty((T, hkv, D), device=DEV, dtype=dt)
        v = torch.empty((T, hkv, D), device=DEV, dtype=dt)
    for x in ([] if decode else [q]) + [k, v]:
        for t in range(0, T, 1 << 18):  # in pieces: the fp32 draw of 1M tokens is large
            piece = randn((min(T, t + (1 << 18)) - t, x.shape[1], D))
            if x is k:
                piece += off[ids[t:t + (1 << 18)]]
            x[t:t + (1 << 18)] = piece
    if decode:
        q.copy_(randn(q.shape))
    dout = randn((T, hq, D), dt) if "train" in case["kind"] else None
    cu = torch.tensor([0] + lens, dtype=torch.int64).cumsum(0).to(torch.int32)
    return {"q": q, "k": k, "v": v, "dout": dout, "cu": cu}


def prepare(case, seed):
    s = _inputs(case, seed)
    s["kind"], s["B"], s["topk"] = case["kind"], case["block"], case["topk"]
    # a decode loop keeps the cache's block means
    s["kbar"] = binding.pool(s["k"], s["cu"], s["B"]) if case["kind"] == "decode" else None
    return s


def run(s):
    q, k, v, cu, kind = s["q"], s["k"], s["v"], s["cu"], s["kind"]
    if "decode" in kind:
        out, lse = binding.decode(q, k, v, cu, s["B"], s["topk"], kbar=s["kbar"])
        return {"out": out, "lse": lse}
    if kind.startswith("full"):
        out, lse = binding.dense_forward(q, k, v, cu)
    else:
        out, lse = binding.forward(q, k, v, cu, s["B"], s["topk"])
    r = {"out": out, "lse": lse}
    if kind == "train":
        r["dq"], r["dk"], r["dv"] = binding.backward(q, k, v, cu, s["B"], s["topk"], out, lse,
                                                     s["dout"])
    elif kind == "full_train":
        r["dq"], r["dk"], r["dv"] = binding.dense_backward(q, k, v, cu, out, lse, s["dout"])
    return r


# --------------------------------------------------------------------- work
def work(case):
    """Each input once and each output once; 4 D operations per attended
    (query, key) pair forward and 10 D backward, 2 D per gate score."""
    lens, hq, hkv, B, k = _lens(case), case["hq"], case["hkv"], case["block"], case["topk"]
    T, G, el = sum(lens), hq // hkv, 4 if case["dtype"] == "f32" else 2
    pairs = scores = 0
    if "decode" in case["kind"]:
        keys = 0.0  # key rows read, per kv-head
        for L in lens:
            c = (L - 1) // B if B else 0
            if not B or c < k:
                pairs += L
                keys += L
            else:
                # blocks that some head of the group selects, on average over
                # independent choices, and the current block
                last = L - c * B
                pairs += (k - 1) * B + last
                keys += c * (1.0 - (1.0 - (k - 1) / c) ** G) * B + last
                scores += c
        b = 2 * el * keys * hkv * D + 2 * el * len(lens) * hq * D + 4 * len(lens) * hq
        if case["kind"] == "decode":
            b += 4 * sum(-(-L // B) for L in lens) * hkv * D
        elif case["kind"] == "decode_fresh":
            b += el * max(0.0, T - keys) * hkv * D  # the means need every key
        return {"bytes": b, "flops": (4 * pairs + 2 * scores) * hq * D}
    for L in lens:
        if not B:
            pairs += L * (L + 1) // 2
            continue
        for c in range(-(-L // B)):
            m = min(L, (c + 1) * B) - c * B
            pairs += m * (m + 1) // 2 + m * B * min(k - 1, c)
            if c > k - 1:
                scores += m * c
    b = el * T * D * (2 * hq + 2 * hkv) + 4 * T * hq
    f = (4 * pairs + 2 * scores) * hq * D
    if "train" in case["kind"]:
        b += el * T * D * (2 * hq + 2 * hkv)  # dout in; dq, dk, dv out
        f += 10 * pairs * hq * D
    return {"bytes": b, "flops": f}


def tolerance(case):
    # measured against exact(): fp32 out 3e-7, lse 5e-8; bf16 out 2.4e-3, gradients 3.0e-3
    if case["dtype"] == "f32":
        return {"rel": 2e-6}
    return {"rel": 1e-2}


# -------------------------------------------------------------------- exact
def _selected(qh, kbar, c, topk):
    """[rows, blocks]: the kept past blocks and the current one; rows of qh at
    current blocks c."""
    n = kbar.shape[0]
    j = torch.arange(n, device=DEV)
    past = j[None, :] < c[:, None]
    s = (qh @ kbar.T).masked_fill(~past, -math.inf)
    keep = torch.zeros_like(past)
    if topk > 1:
        keep.scatter_(1, s.topk(min(topk - 1, n), dim=1).indices, True)
    keep &= past
    keep[torch.arange(len(c), device=DEV), c] = True
    return keep


def exact(case, seed):
    lens, hq, hkv, B, topk = _lens(case), case["hq"], case["hkv"], case["block"], case["topk"]
    decode, train = "decode" in case["kind"], "train" in case["kind"]
    if not decode and hq * sum(L * L for L in lens) > 2.5e11:
        return None
    s = _inputs(case, seed)
    q, k, v, dout = s["q"], s["k"], s["v"], s["dout"]
    G, f64 = hq // hkv, torch.float64
    out = torch.zeros(q.shape, device=DEV, dtype=f64)
    lse = torch.zeros((hq, q.shape[0]), device=DEV, dtype=f64)
    dq = torch.zeros(q.shape, device=DEV, dtype=f64) if train else None
    dk = torch.zeros(k.shape, device=DEV, dtype=f64) if train else None
    dv = torch.zeros(v.shape, device=DEV, dtype=f64) if train else None
    t0 = 0
    for i, L in enumerate(lens):
        Bs = B or L
        blk = torch.arange(L, device=DEV) // Bs
        for g in range(hkv):
            kd, vd = k[t0:t0 + L, g].to(f64), v[t0:t0 + L, g].to(f64)
            kbar = torch.stack([x.mean(0) for x in kd.split(Bs)])
            for h in range(g * G, (g + 1) * G):
                step = max(1, (1 << 26) // L)
                for r0 in range(L - 1 if decode else 0, L, step):
                    r1 = min(L, r0 + step)
                    at = slice(i, i + 1) if decode else slice(t0 + r0, t0 + r1)
                    qh = q[at, h].to(f64)
                    pos = torch.arange(r0, r1, device=DEV)
                    keep = _selected(qh, kbar, pos // Bs, topk or 1)
                    see = keep[:, blk[:r1]] & (torch.arange(r1, device=DEV)[None] <= pos[:, None])
                    z = (qh @ kd[:r1].T).mul_(SCALE).masked_fill_(~see, -math.inf)
                    m = torch.logsumexp(z, 1)
                    p = z.sub_(m[:, None]).exp_()
                    out[at, h] = p @ vd[:r1]
                    lse[h, at] = m
                    if train:
                        do = dout[at, h].to(f64)
                        dv[t0:t0 + r1, g] += p.T @ do
                        dp = do @ vd[:r1].T
                        ds = dp.sub_((p * dp).sum(1, keepdim=True)).mul_(p).mul_(SCALE)
                        dq[at, h] = ds @ kd[:r1]
                        dk[t0:t0 + r1, g] += ds.T @ qh
        t0 += L
    r = {"out": out, "lse": lse}
    if train:
        r.update(dq=dq, dk=dk, dv=dv)
    return r
