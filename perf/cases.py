"""Performance cases of the hybrid-block decode path.

Each case is what a serving program asks of this library while decoding: a
full-attention layer with its token selection, a sparse layer, or a whole
block step (the full layer and the sparse layers that reuse its cache and
selection), through ``hs2.HybridBlock``.

A case holds
  kind      "step" (full layer + n_sparse sparse layers), "full" (the full
            layer and its selection) or "sparse" (one sparse layer)
  kv        "bf16" or "e4m3" (bytes with one scale per KV head)
  layout    of the cache: "record" (K and V of a token side by side),
            "split" (two [B, Hkv, Lmax, D] tensors) or "token" (two
            [B, Lmax, Hkv, D] tensors)
  batch, n_queries (C), n_q_heads, n_kv_heads, head_dim
  ctx, ctx_min   lengths: uniform in [ctx_min, ctx], or ctx when ctx_min is 0
  cap       cache capacity per sequence
  k, window, block (0: token-level selection)
  n_sparse  sparse layers of a step
  extras    sparse layers with per-head sinks and output gates
  needles   planted keys per sequence that the selection has to find

Queries, keys and values are N(0, 1) rounded to bf16, as everywhere in this
repository; an E4M3 cache is the same values at max|x| / 448 per KV head.
"""
import math

import torch

from paper_2609_26368_amd import hs2

E4M3_MAX = 448.0
MAX_ROWS = 128  # query rows per KV head the library serves


def _case(name, kind, kv, layout, batch, n_queries, heads, head_dim, ctx, budget, n_sparse=0, ctx_min=0, cap=0,
          block=0, extras=False, needles=0):
    c = {"kind": kind, "kv": kv, "layout": layout, "batch": batch, "n_queries": n_queries, "n_q_heads": heads[0],
         "n_kv_heads": heads[1], "head_dim": head_dim, "ctx": ctx, "ctx_min": ctx_min, "cap": cap or ctx,
         "k": budget[0], "window": budget[1], "block": block, "n_sparse": n_sparse, "extras": extras,
         "needles": needles}
    return {"name": name, **c} if name else c


def listed():
    return [
        # one short sequence: the smallest step, where launches and latency count
        _case("step_4k", "step", "bf16", "record", 1, 1, (16, 2), 128, 4096, (256, 64), 1),
        # a single 32K sequence, the ordinary interactive decode
        _case("step_32k", "step", "bf16", "record", 1, 1, (32, 4), 128, 32768, (2048, 128), 3),
        # a serving batch of many short and medium sequences, every length its own
        _case("step_batch64_ragged", "step", "bf16", "split", 64, 1, (32, 8), 128, 12000, (512, 128), 3, ctx_min=1000),
        # long ragged sequences with tokens that must be found, on the compressed cache
        _case("step_ragged_e4m3", "step", "e4m3", "record", 8, 1, (32, 4), 128, 131072, (2048, 128), 3,
              ctx_min=16384, needles=16),
        # the same batch on the bf16 cache: its full layer and the selection alone
        _case("full_ragged", "full", "bf16", "record", 8, 1, (32, 4), 128, 131072, (2048, 128), ctx_min=16384,
              needles=16),
        # verification of 8 drafted tokens per sequence at 128K, both cache formats
        _case("full_chunk8", "full", "bf16", "record", 4, 8, (32, 4), 128, 131072, (4096, 256)),
        _case("full_chunk8_e4m3", "full", "e4m3", "record", 4, 8, (32, 4), 128, 131072, (4096, 256)),
        # a sparse layer of that verification, with its sinks and gates
        _case("sparse_chunk8", "sparse", "bf16", "record", 4, 8, (32, 4), 128, 131072, (4096, 256), extras=True),
        # the longest contexts: 512K tokens, the largest case
        _case("step_512k", "step", "bf16", "record", 2, 1, (64, 8), 128, 524288, (8192, 512), 3),
        # the paper's own head layout (MQA 64/1, head dim 256, 1024 + 128 tokens) and cache format
        _case("step_mqa256_e4m3", "step", "e4m3", "record", 8, 1, (64, 1), 256, 131072, (1024, 128), 3, extras=True),
        # the same heads verifying 2 drafted tokens on a bf16 cache
        _case("step_mqa256_chunk2", "step", "bf16", "record", 4, 2, (64, 1), 256, 131072, (1024, 128), 3),
        # odd sizes throughout, token-major cache with room to grow, block-level selection
        _case("full_blocks_odd", "full", "bf16", "token", 5, 3, (24, 4), 128, 20011, (1024, 101), ctx_min=5003,
              cap=21000, block=64),
    ]


def _pow2(x):
    return 1 << (x - 1).bit_length()


def draw(rng):
    """One more case: any head layout the library serves, 1K to 512K tokens, batch 1 to 64, at most half the
    largest listed case's cache."""
    while True:
        kind = rng.choice(["step", "step", "full", "sparse"])
        kv = rng.choice(["bf16", "e4m3"])
        hd = rng.choice([128, 128, 256])
        g = rng.choice([1, 2, 3, 4, 5, 6, 8, 8, 12, 16, 32, 64])
        hkv = rng.choice([1, 2, 4, 8])
        nq = rng.choice([1, 1, 1, 2, 3, 4, 8, 16])
        if nq * _pow2(g) > MAX_ROWS:
            continue
        ctx = int(2 ** rng.uniform(10, 19)) | rng.choice([0, 1])
        batch = int(2 ** rng.uniform(0, 6))
        record = 2 * hd * (2 if kv == "bf16" else 1)
        cap = ctx + rng.choice([0, 0, 7, ctx // 16])
        k = min(int(2 ** rng.uniform(6, 13)), ctx // 2)
        window = rng.choice([0, 64, 101, 128, 256, 512])
        n_sparse = rng.choice([1, 2, 3]) if kind == "step" else 0
        block = 64 if kind == "full" and kv == "bf16" and rng.random() < 0.4 else 0
        if block:
            k = max(block, k // block * block)
        rows = batch * hkv * nq
        if batch * hkv * cap * record > 2.2e9 or rows * cap * 4 > 2.5e8:
            continue
        if rows * (k + window) * record * max(1, n_sparse) > 1e9:
            continue
        # a row whose threshold falls on a near-tie may list another token and shift the slots after it: the
        # selection itself is an output only where that is a small share of all rows
        if kind == "full" and rows < 32:
            continue
        ctx_min = rng.choice([0, ctx // 8, ctx // 2]) if batch > 1 else 0
        return _case("", kind, kv, rng.choice(["record", "record", "split", "token"]), batch, nq, (g * hkv, hkv), hd,
                     ctx, (k, window), n_sparse, ctx_min=max(ctx_min, 64) if ctx_min else 0, cap=cap, block=block,
                     extras=kind != "full" and rng.random() < 0.5, needles=rng.choice([0, 0, 16]))


# ------------------------------------------------------------------ inputs
def _normal(gen, *shape):
    return torch.randn(shape, dtype=torch.float32, device="cuda", generator=gen).to(torch.bfloat16)


def _lengths(c, seed):
    gen = torch.Generator().manual_seed(seed)
    if not c["ctx_min"]:
        return [c["ctx"]] * c["batch"]
    return torch.randint(c["ctx_min"], c["ctx"] + 1, (c["batch"],), generator=gen).tolist()


def _select(scores, n, k, pos, window, slots, block=0):
    """Selected tokens of one row, ascending, -1 padded: the k best of the n candidates (score descending, lower
    index first), or the k / block best blocks, then the window."""
    dev = scores.device
    if block:
        nb = (n + block - 1) // block
        pad = torch.zeros(nb * block, dtype=scores.dtype, device=dev)
        pad[:n] = scores[:n]
        order = torch.sort(pad.view(nb, block).sum(1).float(), descending=True, stable=True).indices
        blocks = order[: k // block]
        top = (blocks[:, None] * block + torch.arange(block, device=dev)).reshape(-1)
        top = top[top < n]
    else:
        top = torch.sort(scores[:n].float(), descending=True, stable=True).indices[:k]
    row = torch.cat([torch.sort(top).values, torch.arange(max(0, pos - window + 1), pos + 1, device=dev)])
    return torch.cat([row, torch.full((slots - row.numel(),), -1, dtype=row.dtype, device=dev)]).int()


def prepare(case, seed):
    """What a serving program holds before the call: the queries of each layer, the cache with its lengths, a
    block handle with its workspace and, for a sparse layer, the selection that the full layer left."""
    c = case
    B, C, Hq, Hkv, D, cap = (c[n] for n in ("batch", "n_queries", "n_q_heads", "n_kv_heads", "head_dim", "cap"))
    gen = torch.Generator(device="cuda").manual_seed(seed)
    lens = _lengths(c, seed)
    q = [_normal(gen, B, C, Hq, D) for _ in range(1 + (c["n_sparse"] if c["kind"] == "step" else 0))]
    if c["layout"] == "record":
        kv = torch.empty(B, Hkv, cap, 2 * D, dtype=torch.bfloat16, device="cuda")
        K, V = kv[..., :D], kv[..., D:]
    elif c["layout"] == "split":
        K, V = (torch.empty(B, Hkv, cap, D, dtype=torch.bfloat16, device="cuda") for _ in range(2))
    else:
        K, V = (torch.empty(B, cap, Hkv, D, dtype=torch.bfloat16, device="cuda").transpose(1, 2) for _ in range(2))
    for b in range(B):
        for X in (K, V):
            X[b] = _normal(gen, Hkv, cap, D)
        if c["needles"]:  # keys along the mean query of their KV head, at about four times its length
            hi = max(1, lens[b] - c["window"] - C)
            at = torch.randint(0, hi, (c["needles"],), device="cuda", generator=gen)
            mean = q[0][b].float().view(C, Hkv, Hq // Hkv, D).mean(dim=(0, 2))
            K[b][:, at] = (4.0 * math.sqrt(D) * mean / mean.norm(dim=1, keepdim=True)).to(torch.bfloat16)[:, None]
    scales = None
    if c["kv"] == "e4m3":
        def quantise(X):
            scale = X.abs().amax(dim=(0, 2, 3)).float() / E4M3_MAX
            X8 = torch.empty(X.shape, dtype=torch.uint8, device="cuda")
            for b in range(B):
                x = (X[b].float() / scale[:, None, None]).clamp(-E4M3_MAX, E4M3_MAX)
                X8[b] = x.to(torch.float8_e4m3fn).view(torch.uint8)
            return X8, scale
        (K8, ks), (V8, vs) = quantise(K), quantise(V)
        scales = (ks, vs)
        if c["layout"] == "record":
            kv = torch.cat([K8, V8], dim=3)
            K, V = kv[..., :D], kv[..., D:]
        elif c["layout"] == "split":
            K, V = K8, V8
        else:
            K, V = (X.transpose(1, 2).contiguous().transpose(1, 2) for X in (K8, V8))
    sink = gate = idx = None
    if c["extras"]:
        sink = torch.randn(Hq, device="cuda", generator=gen)
        gate = _normal(gen, B, C, Hq, D)
    slots = c["k"] + c["window"]
    if c["kind"] == "sparse":
        # a chunk's queries choose largely on their own (a tenth of the variance in common)
        rows = []
        for b in range(B):
            for _ in range(Hkv):
                own = torch.randn(C, cap, device="cuda", generator=gen)
                s = 0.95 * own + 0.31 * torch.randn(cap, device="cuda", generator=gen)
                for j in range(C):
                    pos = lens[b] - C + j
                    rows.append(_select(s[j], max(0, pos - c["window"] + 1), c["k"], pos, c["window"], slots))
        idx = torch.stack(rows).view(B, Hkv, C, slots)
    block = hs2.HybridBlock(B, C, Hq, Hkv, D, cap, c["k"], c["window"], kv_strides=tuple(K.stride()[:3]))
    return {"case": c, "block": block, "q": q, "K": K, "V": V, "lens": torch.tensor(lens, dtype=torch.int32, device="cuda"),
            "scales": scales, "sink": sink, "gate": gate, "idx": idx}


def run(state):
    """One call as a decode loop makes it.  A step's selection goes from its full layer to its sparse layers, whose
    outputs come back."""
    s, c, block = state, state["case"], state["block"]
    K, V, lens = s["K"], s["V"], s["lens"]
    extra = {"sink": s["sink"], "gate": s["gate"], "kv_scales": s["scales"]}
    if c["kind"] == "sparse":
        return block.sparse(s["q"][0], K, V, lens, s["idx"], **extra)
    out, idx = block.full(s["q"][0], K, V, lens, kv_scales=s["scales"], block=c["block"] or None)
    if c["kind"] == "full":
        return out, idx
    return [out] + [block.sparse(q, K, V, lens, idx, **extra) for q in s["q"][1:]]


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    """Full layer: the cache once, queries, output and the selection; Q.K and P.V over every token.  Sparse layer:
    the cache rows that its rows select (a chunk's queries share rows as independent picks do), the selection,
    queries and output; Q.K and P.V over every slot."""
    c = case
    B, C, Hq, Hkv, D = (c[n] for n in ("batch", "n_queries", "n_q_heads", "n_kv_heads", "head_dim"))
    record = 2 * D * (2 if c["kv"] == "bf16" else 1)
    mean = (c["ctx_min"] + c["ctx"]) / 2 if c["ctx_min"] else c["ctx"]
    slots = min(c["k"] + c["window"], mean)
    io = 2 * B * C * Hq * D * 2
    picks = B * Hkv * C * slots * 4
    n = max(1.0, mean - c["window"])
    unique = min(mean, c["window"] + C - 1 + n * (1 - (1 - min(1.0, c["k"] / n)) ** C))
    sparse = {"bytes": B * Hkv * unique * record + picks + io + (io / 2 if c["extras"] else 0),
              "flops": 4.0 * B * C * Hq * D * slots}
    full = {"bytes": B * Hkv * mean * record + picks + io, "flops": 4.0 * B * C * Hq * D * mean}
    if c["kind"] == "sparse":
        return sparse
    if c["kind"] == "full":
        return full
    return {m: full[m] + c["n_sparse"] * sparse[m] for m in full}


def tolerance(case):
    """bf16 outputs and probabilities: the same path with its sums split otherwise is up to 3.1e-3 away, an element up
    to 0.018 of the root mean square; four times that.  The 32-bit scores of two tokens at the selection's threshold may fall
    either way: a few of the rows then differ from that slot on, and a step's sparse outputs by one token's value."""
    tol = {"rel": 1.2e-2, "max": 0.07}
    if case["kind"] == "full":
        tol["differ"] = 0.01
    if case["kind"] == "step" and case["ctx"] > 16384:
        tol = {"rel": 2e-2, "max": 0.4}
    return tol


# ------------------------------------------------------------------ 64-bit values
def _exact_attention(q, k, v, scale, causal_pos=None, sink=None):
    """q [R, D], k and v [T, D] float64: outputs [R, D] and probabilities [R, T]; row r sees tokens up to
    causal_pos[r]; sink [R] joins the normaliser."""
    s = (q @ k.t()) * scale
    if causal_pos is not None:
        s.masked_fill_(torch.arange(s.shape[1], device=s.device)[None] > causal_pos[:, None], -math.inf)
    m = s.amax(dim=1, keepdim=True)
    if sink is not None:
        m = torch.maximum(m, sink[:, None])
    p = torch.exp(s - m)
    z = p.sum(dim=1, keepdim=True)
    if sink is not None:
        z = z + torch.exp(sink[:, None] - m)
    p /= z
    return p @ v, p


def exact(case, seed):
    """run()'s outputs in 64-bit torch.  A step's sparse outputs have no such value when a row's selection hangs on
    two scores that 32-bit arithmetic cannot tell apart."""
    c = case
    st = prepare(c, seed)
    B, C, Hq, Hkv, D = (c[n] for n in ("batch", "n_queries", "n_q_heads", "n_kv_heads", "head_dim"))
    G, slots, scale = Hq // Hkv, c["k"] + c["window"], 1.0 / math.sqrt(c["head_dim"])
    lens = st["lens"].tolist()

    def values(X, b, g, which, rows):
        x = X[b, g][rows]
        if st["scales"] is None:
            return x.double()
        return x.contiguous().view(torch.float8_e4m3fn).float().double() * st["scales"][which][g].double()

    def sparse(q, idx):
        out = torch.empty(B, C, Hq, D, dtype=torch.float64, device="cuda")
        for b in range(B):
            for g in range(Hkv):
                h = slice(g * G, (g + 1) * G)
                sink = st["sink"][h].double() if st["sink"] is not None else None
                for j in range(C):
                    t = idx[b, g, j]
                    t = t[t >= 0].long()
                    out[b, j, h] = _exact_attention(q[b, j, h].double(), values(st["K"], b, g, 0, t),
                                                    values(st["V"], b, g, 1, t), scale, sink=sink)[0]
        return out * torch.sigmoid(st["gate"].double()) if st["gate"] is not None else out

    if c["kind"] == "sparse":
        return sparse(st["q"][0], st["idx"])
    out = torch.empty(B, C, Hq, D, dtype=torch.float64, device="cuda")
    idx = torch.empty(B, Hkv, C, slots, dtype=torch.int32, device="cuda")
    near = False
    for b in range(B):
        L = lens[b]
        pos = torch.arange(L - C, L, device="cuda")
        for g in range(Hkv):
            h = slice(g * G, (g + 1) * G)
            t = slice(0, L)
            o, p = _exact_attention(st["q"][0][b, :, h].reshape(C * G, D).double(), values(st["K"], b, g, 0, t),
                                    values(st["V"], b, g, 1, t), scale, pos.repeat_interleave(G))
            out[b, :, h] = o.view(C, G, D)
            pooled = p.view(C, G, L).sum(1)
            for j in range(C):
                n = max(0, L - C + j - c["window"] + 1)
                idx[b, g, j] = _select(pooled[j], n, c["k"], L - C + j, c["window"], slots, c["block"])
                if c["kind"] == "step" and 0 < c["k"] < n:
                    best = torch.topk(pooled[j, :n], c["k"] + 1).values
                    near = near or bool((best[-2] - best[-1]) < 2e-6 * best[-2])
    if c["kind"] == "full":
        return out, idx
    return [out] + [None if near else sparse(q, idx) for q in st["q"][1:]]
