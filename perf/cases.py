"""The work that this library is timed on, through its public entry points (paper_2601_21896_amd.binding).

A case is a dict of plain sizes and options.  `listed()` names the fixed ones, `draw(rng)` gives another of the same
ranges, `prepare` makes on the GPU what a caller holds before the call (activations, cache slabs, head weights, output
buffers, workspace, the argument struct), `run` is one call and its outputs.

The path is an inference step of one or more attention layers: score tokens with the salience head, keep the top `keep`
of the cache, compact K/V to them, attend from the chunk over retained + chunk.  Kinds:
  step      - pafu_step: one layer.  mode "single" scores cache and chunk and selects on the fresh scores; "rollout"
              scores the chunk only, selects on the stored list and appends the chunk behind the retained rows.
  layers    - pafu_step_layers (every layer selects for itself) or pafu_step_layers_shared (one index list for all).
  attention - the attention call alone: over a compacted cache, or through an index list ("gather").
  sse       - pafu_sse_score, the teacher-side score the salience head is trained on.
  quantise  - the two directions of the 8-bit cache format over a whole cache.
`exact` is what a call returns in 64 bits, in plain torch.

Values follow workloads.py: N(0,1) features, Q, K, V; a per-channel key scale from U[0.5, 2]; N(0, 0.02^2) head weights;
a tenth of the cached tokens salient (+2 on every feature, or a higher stored score).
"""

from __future__ import annotations

import math

import torch

from paper_2601_21896_amd import binding as B

DEV = "cuda:0"
BF = torch.bfloat16
K_SCALE_LOG2, V_SCALE_LOG2 = -5, -6  # 8-bit cache: |K| <= 14 and |V| <= 7 are representable
MOST_FLOPS = 1.5e13                  # no drawn case is above the largest listed one (30 rollout layers)
MOST_BYTES = 1.4e10


# ------------------------------------------------------------------------------------------------ the cases
def _step(name, mode, heads, head_dim, cached, chunk, keep, **kw):
    c = {"name": name, "kind": "step", "mode": mode, "heads": heads, "head_dim": head_dim, "cached": cached,
         "chunk": chunk, "keep": keep, "block": chunk, "hidden": 256, "outputs": 1, "segments": 1, "bias": False,
         "features": "bf16", "kv": "bf16", "out": "bf16", "pinned": 0, "layers": 1, "shared": False}
    c.update(kw)
    return c


def listed():
    return [
        # the smallest step: two heads of 64, one 64-token frame against four, fp32 features; launches and latency
        _step("step_tiny", "single", 2, 64, 256, 64, 128, hidden=32, features="fp32"),
        # the headline: a Wan-1.3B layer, 21 cached frames of 1560 tokens, a 3-frame chunk, half of the cache kept
        _step("step_1p3b", "single", 12, 128, 32760, 4680, 16380),
        # steady state of a rollout at that layer: 8 frames kept, the chunk appended
        _step("rollout_1p3b", "rollout", 12, 128, 17160, 4680, 12480),
        # the same with the 8-bit cache
        _step("rollout_1p3b_e4m3", "rollout", 12, 128, 17160, 4680, 12480, kv="e4m3"),
        # the paper's inference setting: 3 frames kept, first frame pinned, head over [Q | K | V] with 12 outputs
        _step("rollout_paper_head", "rollout", 12, 128, 9360, 4680, 4680, hidden=1024, outputs=12, segments=3,
              pinned=1560),
        # a Wan-14B layer at 720p: 40 heads, 21 frames of 3600 tokens
        _step("rollout_14b", "rollout", 40, 128, 75600, 10800, 22680, hidden=512),
        # all 30 layers of a Wan-1.3B model, one index list for all of them (the largest case)
        _step("layers_30_shared", "rollout", 12, 128, 17160, 4680, 12480, kind="layers", layers=30, shared=True),
        # several independent layers at odd sizes: head dim 64, frame-wise block mask, biases, averaged outputs
        _step("layers_ragged", "single", 8, 64, 6007, 1203, 2999, kind="layers", layers=6, block=401, hidden=128,
              outputs=4, bias=True, out="fp32"),
        # a one-frame chunk over a long cache: few queries, many keys
        {"name": "attention_frame", "kind": "attention", "gather": False, "heads": 12, "head_dim": 128,
         "cached": 16380, "keep": 16380, "chunk": 1560, "block": 1560, "kv": "bf16", "out": "bf16"},
        # attention through an index list over the uncompacted cache, ragged
        {"name": "attention_gather", "kind": "attention", "gather": True, "heads": 12, "head_dim": 128,
         "cached": 32760, "keep": 8191, "chunk": 3121, "block": 1041, "kv": "bf16", "out": "bf16"},
        # the teacher score of a 21-frame clip, blocks of 3 frames
        {"name": "sse_teacher", "kind": "sse", "heads": 12, "head_dim": 128, "tokens": 32760, "block": 4680},
        # a Wan-1.3B cache to 8-bit codes and back
        {"name": "cache_to_e4m3_and_back", "kind": "quantise", "heads": 12, "head_dim": 128, "tokens": 32760},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_once(rng):
    kind = rng.choice(["step"] * 5 + ["layers"] * 2 + ["attention"] * 3 + ["sse", "quantise"])
    head_dim = rng.choice([128, 128, 128, 64])
    heads = rng.choice([2, 5, 8, 12, 12, 16, 24, 40])
    if kind == "sse":
        tokens = _log_int(rng, 500, 40000)
        return {"kind": kind, "heads": heads, "head_dim": head_dim, "tokens": tokens,
                "block": max(1, tokens // rng.choice([1, 2, 3, 7, 7, 21]))}
    if kind == "quantise":
        return {"kind": kind, "heads": heads, "head_dim": head_dim, "tokens": _log_int(rng, 200, 80000)}
    chunk = _log_int(rng, 48, 10800)
    cached = _log_int(rng, 256, 80000)
    keep = max(1, int(cached * rng.choice([rng.uniform(0.05, 1.0)] * 7 + [1.25])))  # 1.25: nothing to evict yet
    block = rng.choice([chunk, chunk, max(1, chunk // 3)])
    if kind == "attention":
        gather = rng.random() < 0.4
        return {"kind": kind, "gather": gather, "heads": heads, "head_dim": head_dim, "cached": cached,
                "keep": min(keep, cached), "chunk": chunk, "block": block,
                "kv": "e4m3" if head_dim == 128 and not gather and rng.random() < 0.3 else "bf16",
                "out": rng.choice(["bf16", "bf16", "fp32"])}
    kw = {"kind": kind, "block": block, "hidden": rng.choice([128, 256, 256, 512, 1024]),
          "outputs": rng.choice([1, 1, 12]), "segments": rng.choice([1, 1, 1, 3]), "bias": rng.random() < 0.3,
          "pinned": rng.choice([0, 0, min(cached // 4, chunk // 3)]), "out": rng.choice(["bf16", "bf16", "fp32"])}
    mode = rng.choice(["single", "rollout", "rollout"])
    if kind == "layers":
        kw["layers"], kw["shared"] = _log_int(rng, 2, 40), rng.random() < 0.5
    if head_dim == 128 and rng.random() < 0.25:
        kw["kv"] = "e4m3"
    if kind == "step" and rng.random() < 0.2:  # the small end: fp32 features go with small models
        heads, head_dim = rng.choice([1, 2, 4]), 64
        cached, chunk = _log_int(rng, 64, 1500), _log_int(rng, 16, 300)
        kw.update(block=chunk, hidden=rng.choice([32, 64]), features="fp32", kv="bf16", segments=1, pinned=0)
        keep = max(1, int(cached * rng.uniform(0.1, 1.0)))
    c = _step("", mode, heads, head_dim, cached, chunk, keep, **kw)
    del c["name"]
    return c


def draw(rng):
    while True:
        c = _draw_once(rng)
        w = work(c)
        if w["flops"] <= MOST_FLOPS and w["bytes"] <= MOST_BYTES:
            return c


# ------------------------------------------------------------------------------------------------ inputs
class _Maker:
    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(seed)

    def normal(self, *shape):
        return torch.randn(*shape, device=DEV, generator=self.g)

    def uniform(self, *shape):
        return torch.rand(*shape, device=DEV, generator=self.g)

    def tokens(self, rows, width, scale=None, dtype=BF):
        """[rows, width] N(0,1) (times a per-channel scale)."""
        out = torch.empty(rows, width, device=DEV, dtype=dtype)
        for r in range(0, rows, 16384):  # in pieces: the fp32 draw of a large tensor is not kept beside it
            m = min(16384, rows - r)
            x = self.normal(m, width)
            out[r:r + m] = x if scale is None else x * scale
        return out

    def salient(self, rows):
        return torch.randperm(rows, device=DEV, generator=self.g)[:rows // 10]


def _bytes(n):
    return torch.empty(max(int(n), 16), dtype=torch.uint8, device=DEV)


def _codes(K, V):
    """The 8-bit rows of a K/V pair."""
    rows, N, D = K.shape
    Kq, Vq = (torch.empty(rows, N * D, dtype=torch.uint8, device=DEV) for _ in range(2))
    B.pafu_quantize_kv(K, V, K_SCALE_LOG2, V_SCALE_LOG2, Kq, Vq)
    return Kq, Vq


def _prepare_layers(c, seed):
    mk = _Maker(seed)
    N, D, n, Lc, k, layers = c["heads"], c["head_dim"], c["cached"], c["chunk"], c["keep"], c["layers"]
    H, kept = N * D, min(c["keep"], c["cached"])
    single, e4m3 = c["mode"] == "single", c["kv"] == "e4m3"
    xdt = torch.float32 if c["features"] == "fp32" else BF
    odt = torch.float32 if c["out"] == "fp32" else BF
    rows_out = kept + (Lc if e4m3 or not single else 0)
    kv_shape, kv_dt = ((layers, rows_out, H), torch.uint8) if e4m3 else ((layers, rows_out, N, D), BF)
    out = {"O": torch.empty(layers, Lc, N, D, device=DEV, dtype=odt),
           "K": torch.empty(kv_shape, device=DEV, dtype=kv_dt), "V": torch.empty(kv_shape, device=DEV, dtype=kv_dt)}
    heads = 1 if c["shared"] else layers  # layers that score and select for themselves
    out["ids"] = torch.empty(heads, kept, dtype=torch.int32, device=DEV)
    # the score list: retained scores, in a rollout with the chunk's behind them
    out["SL"] = torch.empty(heads, kept + (0 if single else Lc), device=DEV)
    if single:
        # (every layer's score list starts at a 16-byte boundary)
        out["scores"] = torch.empty(heads, (n + Lc + 3) // 4 * 4, device=DEV)[:, :n + Lc]
    index_layer = layers - 1 if c["shared"] else None
    args, given = [], []
    for l in range(layers):
        s = 0 if c["shared"] else l
        scale = mk.uniform(H) * 1.5 + 0.5
        Kc, Vc = mk.tokens(n, H, scale).view(n, N, D), mk.tokens(n, H).view(n, N, D)
        if e4m3:
            Kc, Vc = _codes(Kc, Vc)
        Q = mk.tokens(Lc, H).view(Lc, N, D)
        Kn, Vn = mk.tokens(Lc, H, scale).view(Lc, N, D), mk.tokens(Lc, H).view(Lc, N, D)
        scores = SL_in = x_cache = b1 = b2 = None
        layer = {"K": Kc, "V": Vc, "Q": Q, "Kn": Kn, "Vn": Vn}
        if index_layer is None or l == index_layer:
            hot = mk.salient(n)
            W1 = (mk.normal(c["hidden"], c["segments"] * H) * 0.02).to(xdt)
            W2 = mk.normal(c["outputs"], c["hidden"]) * 0.02
            if c["bias"]:
                b1, b2 = mk.normal(c["hidden"]) * 0.02, mk.normal(c["outputs"]) * 0.02
            if single:
                xs = [mk.tokens(n + Lc, H, dtype=xdt) for _ in range(c["segments"])]
                for x in xs:
                    x[hot] += 2.0
                x_cache, x_chunk = tuple(x[:n] for x in xs), tuple(x[n:] for x in xs)
                scores = out["scores"][s]
            else:
                x_chunk = tuple(mk.tokens(Lc, H, dtype=xdt) for _ in range(c["segments"]))
                SL_in = mk.normal(n) * 0.15
                SL_in[hot] += 0.5
            layer.update(x_cache=x_cache, x_chunk=x_chunk, W1=W1, b1=b1, W2=W2, b2=b2, SL=SL_in)
        # (with shared indices the other layers' feature, weight and score fields are ignored; they name the last
        # layer's here only because the struct is filled from tensors)
        if c["shared"] and l != index_layer:
            W1, W2, x_chunk = torch.empty(1, H, device=DEV, dtype=xdt), torch.empty(1, 1, device=DEV), (Q.view(Lc, H),)
        a = B.make_step_args(B.PAFU_MODE_SINGLE if single else B.PAFU_MODE_ROLLOUT, N, D, n, Lc, k, c["block"], x_cache,
                             x_chunk, W1, b1, W2, b2, Kc, Vc, SL_in, Q, Kn, Vn, scores, out["ids"][s], out["K"][l],
                             out["V"][l], out["SL"][s], out["O"][l], n_pinned=c["pinned"],
                             kv_dtype=B.PAFU_FP8_E4M3 if e4m3 else B.PAFU_BF16,
                             k_scale_log2=K_SCALE_LOG2 if e4m3 else 0, v_scale_log2=V_SCALE_LOG2 if e4m3 else 0)
        args.append(a)
        given.append(layer)
    ws = _bytes(max(B.pafu_step_workspace_bytes(a) for a in args))
    for a in args:
        a.workspace, a.workspace_bytes = ws.data_ptr(), ws.numel()
    return {"case": c, "args": args, "out": out, "ws": ws, "index_layer": index_layer, "given": given}


def prepare(case, seed):
    c = dict(case)
    if c["kind"] in ("step", "layers"):
        return _prepare_layers(c, seed)
    mk = _Maker(seed)
    N, D = c["heads"], c["head_dim"]
    H = N * D
    scale = mk.uniform(H) * 1.5 + 0.5
    st = {"case": c}
    if c["kind"] == "sse":
        L = c["tokens"]
        st["Q"], st["K"] = mk.tokens(L, H).view(L, N, D), mk.tokens(L, H, scale).view(L, N, D)
        st["out"] = torch.empty(L, device=DEV)
        st["ws"] = _bytes(B.pafu_sse_workspace_bytes(L, N))
    elif c["kind"] == "quantise":
        L = c["tokens"]
        st["K"], st["V"] = mk.tokens(L, H, scale).view(L, N, D), mk.tokens(L, H).view(L, N, D)
        st["Kq"], st["Vq"] = (torch.empty(L, H, dtype=torch.uint8, device=DEV) for _ in range(2))
        st["Kb"], st["Vb"] = torch.empty_like(st["K"]), torch.empty_like(st["V"])
    else:
        Lc, rows = c["chunk"], c["cached"] if c["gather"] else c["keep"]
        st["Q"] = mk.tokens(Lc, H).view(Lc, N, D)
        st["K"], st["V"] = mk.tokens(rows, H, scale).view(rows, N, D), mk.tokens(rows, H).view(rows, N, D)
        st["Kn"], st["Vn"] = mk.tokens(Lc, H, scale).view(Lc, N, D), mk.tokens(Lc, H).view(Lc, N, D)
        if c["kv"] == "e4m3":
            st["K"], st["V"] = _codes(st["K"], st["V"])
            st["Kn"], st["Vn"] = _codes(st["Kn"], st["Vn"])
        if c["gather"]:
            keep = torch.randperm(rows, device=DEV, generator=mk.g)[:c["keep"]]
            st["ids"] = torch.sort(keep).values.to(torch.int32)
        st["O"] = torch.empty(Lc, N, D, device=DEV, dtype=torch.float32 if c["out"] == "fp32" else BF)
        st["ws"] = _bytes(B.pafu_attention_workspace_bytes(Lc, N, D))
    return st


# ------------------------------------------------------------------------------------------------ one pass
def run(st):
    c = st["case"]
    kind = c["kind"]
    if kind == "step":
        B.pafu_step(st["args"][0])
        return st["out"]
    if kind == "layers":
        if c["shared"]:
            B.pafu_step_layers_shared(st["args"], st["index_layer"])
        else:
            B.pafu_step_layers(st["args"])
        return st["out"]
    if kind == "sse":
        return B.pafu_sse_score(st["Q"], st["K"], c["block"], st["out"], st["ws"])
    if kind == "quantise":
        B.pafu_quantize_kv(st["K"], st["V"], K_SCALE_LOG2, V_SCALE_LOG2, st["Kq"], st["Vq"])
        B.pafu_dequantize_kv(st["Kq"], st["Vq"], K_SCALE_LOG2, V_SCALE_LOG2, st["Kb"], st["Vb"])
        return [st[x] for x in ("Kq", "Vq", "Kb", "Vb")]
    if c["gather"]:
        return B.pafu_chunk_attention_gather(st["Q"], st["K"], st["V"], st["ids"], c["keep"], st["Kn"], st["Vn"],
                                             c["block"], st["O"], workspace=st["ws"])
    if c["kv"] == "e4m3":
        return B.pafu_chunk_attention_fp8(st["Q"], st["K"], st["V"], c["keep"], st["Kn"], st["Vn"], c["block"],
                                          K_SCALE_LOG2, V_SCALE_LOG2, st["O"], workspace=st["ws"])
    return B.pafu_chunk_attention(st["Q"], st["K"], st["V"], c["keep"], st["Kn"], st["Vn"], c["block"], st["O"],
                                  workspace=st["ws"])


# ------------------------------------------------------------------------------------------------ what it takes
def _visible_pairs(chunk, kept, block):
    """(query, key) pairs of the attention: all retained keys, and the chunk's up to the end of the query's block."""
    own, i = 0, 0
    while i < chunk:
        m = min(block, chunk - i)
        own += m * (i + m)
        i += m
    return chunk * kept + own


def work(c):
    N, D = c["heads"], c["head_dim"]
    H = N * D
    if c["kind"] == "sse":  # two products with the same operands: normalisers, then maxima
        L = c["tokens"]
        return {"bytes": 2 * L * H * 2 + 4 * L, "flops": 2 * 2 * L * L * H}
    if c["kind"] == "quantise":  # bf16 read, codes written; codes read, bf16 written
        return {"bytes": 2 * c["tokens"] * H * (2 + 1 + 1 + 2), "flops": 0}
    Lc = c["chunk"]
    kept = min(c["keep"], c["cached"])
    kvb = 1 if c["kv"] == "e4m3" else 2
    ob = 4 if c["out"] == "fp32" else 2
    flops = 4 * H * _visible_pairs(Lc, kept, c["block"])
    if c["kind"] == "attention":
        return {"bytes": 2 * (kept + Lc) * H * kvb + Lc * H * (2 + ob) + (4 * kept if c["gather"] else 0),
                "flops": flops}
    single = c["mode"] == "single"
    # a layer's cache: retained rows read and written, chunk rows read (and written where they enter the cache)
    rows_out = kept + (Lc if kvb == 1 or not single else 0)
    layer = 2 * H * (kept * kvb + Lc * 2 + rows_out * kvb) + Lc * H * (2 + ob)
    # a scoring layer: features and weights read, scores and indices written, the score list read and compacted
    F, T = c["segments"] * H, Lc + (c["cached"] if single else 0)
    xb = 4 if c["features"] == "fp32" else 2
    head = (T + c["hidden"]) * F * xb + 4 * T + 4 * kept * 2 + (0 if single else 4 * c["cached"])
    heads = 1 if c["shared"] else c["layers"]
    return {"bytes": layer * c["layers"] + head * heads,
            "flops": flops * c["layers"] + (2 * F * c["hidden"] * T + 2 * c["hidden"] * T) * heads}


def tolerance(c):
    """What another correct implementation at the same precision may differ by.

    Measured against the same formulas in 64 bits on sampled rows: O is off by 2.3e-3 (2-norm) and 1.2e-2 (largest) in
    every case, which is the rounding of the softmax weights and of O to bf16; fp32 scores by 4e-7 and 1.5e-6, the
    teacher score by 3.5e-7 and 6e-7.  Indices, cache rows and codes are whole numbers or copies: they stay the same."""
    if c["kind"] == "quantise":
        return "exact"
    if c["kind"] == "sse":
        return {"rel": 1e-5, "max": 1e-4}
    return {"rel": 1e-2, "max": 5e-2}


# ------------------------------------------------------------------------------------------------ in 64 bits
def _decoded(codes, scale_log2, shape):
    return (codes.view(torch.float8_e4m3fn).double() * 2.0 ** scale_log2).view(shape)


def _encoded(x, scale_log2):
    """(bf16 values are well inside fp32, where the scaling is exact; saturation comes before the cast)"""
    y = (x.float() * 2.0 ** -scale_log2).clamp(-448.0, 448.0)
    return y.to(torch.float8_e4m3fn).view(torch.uint8).view(x.shape[0], -1)


def _attend(Q, K, V, kept, block):
    """softmax(Q K^T / sqrt(D)) V per head; the keys are `kept` retained ones, then the chunk's."""
    Lc, N, D = Q.shape
    out = torch.empty(Lc, N, D, device=DEV, dtype=torch.float64)
    for h in range(N):
        q, k, v = Q[:, h].double(), K[:, h].double().contiguous(), V[:, h].double().contiguous()
        i = 0
        while i < Lc:  # a block of queries sees one prefix of the keys; large ones go in pieces
            seen = kept + min((i // block + 1) * block, Lc)
            m = min(2048, (i // block + 1) * block - i, Lc - i)
            s = (q[i:i + m] @ k[:seen].t()) / math.sqrt(D)
            out[i:i + m, h] = torch.softmax(s, dim=1) @ v[:seen]
            i += m
    return out


def _scored(xs, w):
    parts = []
    for r in range(0, xs[0].shape[0], 8192):
        h = torch.cat([x[r:r + 8192].double() for x in xs], dim=1) @ w["W1"].double().t()
        h = h if w["b1"] is None else h + w["b1"].double()
        o = (h * torch.sigmoid(h)) @ w["W2"].double().t()
        parts.append((o if w["b2"] is None else o + w["b2"].double()).mean(dim=1))
    return torch.cat(parts)


def _exact_layers(c, st):
    """Where the kept tokens follow from scores computed in the call ("single"), two close scores may change places:
    the outputs that such a change moves by a row (indices, cache rows, their scores) are left out there."""
    n, Lc, N, D = c["cached"], c["chunk"], c["heads"], c["head_dim"]
    kept, single, e4m3 = min(c["keep"], n), c["mode"] == "single", c["kv"] == "e4m3"
    out, ids_of, row = {"O": [], "K": [], "V": [], "ids": [], "SL": [], "scores": []}, {}, ("ids", "SL", "scores")
    scoring = [l for l in range(c["layers"]) if st["index_layer"] in (None, l)]
    for l in scoring:
        w = st["given"][l]
        new = _scored(w["x_chunk"], w)
        stored = _scored(w["x_cache"], w) if single else w["SL"].double()
        rank = stored.clone()
        rank[:c["pinned"]] = math.inf
        best = torch.sort(rank, descending=True, stable=True).indices[:kept]
        ids_of[l] = torch.sort(best).values
        out["ids"].append(ids_of[l].to(torch.int32))
        out["SL"].append(stored[ids_of[l]] if single else torch.cat([stored[ids_of[l]], new]))
        out["scores"].append(torch.cat([stored, new]))
    for l, w in enumerate(st["given"]):
        ids = ids_of[scoring[0] if c["shared"] else l]
        K, V, Kn, Vn = w["K"][ids], w["V"][ids], w["Kn"], w["Vn"]
        if e4m3:
            Kn, Vn = _encoded(Kn, K_SCALE_LOG2), _encoded(Vn, V_SCALE_LOG2)
        K, V = torch.cat([K, Kn]), torch.cat([V, Vn])
        rows = kept + (Lc if e4m3 or not single else 0)
        out["K"].append(K[:rows])
        out["V"].append(V[:rows])
        if e4m3:
            K, V = _decoded(K, K_SCALE_LOG2, (-1, N, D)), _decoded(V, V_SCALE_LOG2, (-1, N, D))
        out["O"].append(_attend(w["Q"], K, V, kept, c["block"]))
    out = {k: torch.stack(v) for k, v in out.items()}
    if single:
        return {"O": out["O"], "K": None, "V": None, "ids": None, "SL": None, "scores": out["scores"]}
    del out["scores"]
    return out


def _exact_sse(c, st):
    """Per key the largest weight over the queries of later, the same and earlier blocks, averaged over the heads; the
    score is the mean of the parts that exist (Eq. 4-5)."""
    L, N, D = st["Q"].shape
    block = c["block"]
    starts = list(range(0, L, block))
    total = torch.zeros(L, device=DEV, dtype=torch.float64)
    own = torch.arange(L, device=DEV) // block
    parts = (1 + (own > 0).int() + (own < len(starts) - 1).int()).double()
    for h in range(N):
        k = st["K"][:, h].double().contiguous()
        best = torch.zeros(3, L, device=DEV, dtype=torch.float64)
        for b, lo in enumerate(starts):
            hi = min(lo + block, L)
            for i in range(lo, hi, 2048):  # (a part with no queries stays 0)
                q = st["Q"][i:min(i + 2048, hi), h].double()
                top = torch.softmax((q @ k.t()) / math.sqrt(D), dim=1).amax(dim=0)
                for part, of in enumerate((own < b, own == b, own > b)):
                    best[part] = torch.where(of, torch.maximum(best[part], top), best[part])
        total += best.sum(dim=0)
    return total / N / parts


def exact(case, seed):
    c = dict(case)
    st = prepare(c, seed)
    if c["kind"] in ("step", "layers"):
        return _exact_layers(c, st)
    if c["kind"] == "sse":
        return _exact_sse(c, st)
    if c["kind"] == "quantise":
        Kq, Vq = _encoded(st["K"], K_SCALE_LOG2), _encoded(st["V"], V_SCALE_LOG2)
        shape = st["K"].shape
        return [Kq, Vq, _decoded(Kq, K_SCALE_LOG2, shape), _decoded(Vq, V_SCALE_LOG2, shape)]
    K, V, Kn, Vn = st["K"], st["V"], st["Kn"], st["Vn"]
    if c["gather"]:
        K, V = K[st["ids"].long()], V[st["ids"].long()]
    K, V = torch.cat([K, Kn.view(Kn.shape[0], *K.shape[1:])]), torch.cat([V, Vn.view(Vn.shape[0], *V.shape[1:])])
    if c["kv"] == "e4m3":
        shape = (-1, c["heads"], c["head_dim"])
        K, V = _decoded(K, K_SCALE_LOG2, shape), _decoded(V, V_SCALE_LOG2, shape)
    return _attend(st["Q"], K, V, c["keep"], c["block"])
