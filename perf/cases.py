"""Performance cases: calls of the two reduction stages as an inference program makes them.

A case is one call of a public entry point of `paper_2505_22654_amd.binding`.  `prepare` makes
what the program holds before the call: the layer's tensors, drawn on the GPU by the recipe of
`paper_2505_22654_amd/workloads.py` (clustered patch features, random projections, N(0, 1) decoder
states with a few visual keys nudged towards the query), and the workspace it keeps between calls.
Result tensors are allocated by the call, as they are when they travel on through a model.

Fields of a case
  path     "encode" (stage 1: score, select, assign, merge) or "prune" (stage 2: score, select,
           compact)
  source   "qk": the layer's queries and keys are at hand; "hidden": scored from hidden states and
           projection weights
  dtype    "bf16" or "f32"
  encode:  batch images of `crops` segments of grid_h x grid_w tokens; `mean`: scored by mean
           attention received (no [CLS] row) instead of the [CLS] row; `shallow`: a second,
           shallow-layer pair drives the local scan; `all_keys`: softmax over the whole row
  prune:   batch sequences of prefix + vis + text tokens; layout "dense" (out of place),
           "in_place", or "ragged" (lengths drawn from `lens_seed` below the capacities)
"""
import math
import random

import torch

from paper_2505_22654_amd import binding as vb
from paper_2505_22654_amd import workloads as wl

_TORCH = {"f32": torch.float32, "bf16": torch.bfloat16}


# ------------------------------------------------------------------------------------- the cases
def _encode(name, dtype, batch, crops, grid_h, grid_w, heads, head_dim, win_rows, win_cols,
            keep_global, keep_local, source="qk", mean=False, shallow=False, all_keys=False):
    return {"name": name, "path": "encode", "source": source, "dtype": dtype, "batch": batch,
            "crops": crops, "grid_h": grid_h, "grid_w": grid_w, "mean": mean, "shallow": shallow,
            "all_keys": all_keys, "heads": heads, "head_dim": head_dim, "win_rows": win_rows,
            "win_cols": win_cols, "keep_global": keep_global, "keep_local": keep_local}


def _prune(name, dtype, batch, prefix, vis, text, n_query, q_heads, kv_heads, head_dim, hidden,
           keep, source="qk", layout="dense", all_keys=False, lens_seed=0):
    return {"name": name, "path": "prune", "source": source, "dtype": dtype, "layout": layout,
            "batch": batch, "prefix": prefix, "vis": vis, "text": text, "n_query": n_query,
            "q_heads": q_heads, "kv_heads": kv_heads, "head_dim": head_dim, "hidden": hidden,
            "keep": keep, "all_keys": all_keys, "lens_seed": lens_seed}


def listed():
    return [
        # one 24x24 image in fp32: the smallest call, a single interactive request
        _encode("encode-1x576-f32", "f32", 1, 1, 24, 24, 16, 64, 2, 2, 32, 32),
        # a serving batch of single-crop images at a third of their tokens
        _encode("encode-16x576", "bf16", 16, 1, 24, 24, 16, 64, 4, 4, 96, 96),
        # high-resolution images of five crops each, merged across crops
        _encode("encode-8x5x576", "bf16", 8, 5, 24, 24, 16, 64, 4, 4, 32, 32),
        # an encoder without [CLS] at its largest native resolution: N x N attention
        _encode("encode-mean-16384", "bf16", 1, 1, 128, 128, 16, 80, 8, 8, 2048, 2048, mean=True),
        # the same encoder on two photographs of an odd aspect ratio, with the shallow-layer pair
        _encode("encode-mean-2x45x61", "bf16", 2, 1, 45, 61, 16, 80, 5, 7, 350, 343, mean=True,
                shallow=True),
        # the serving batch scored before its layer has run: hidden states and weights
        _encode("encode-hidden-16x576", "bf16", 16, 1, 24, 24, 16, 64, 4, 4, 64, 64,
                source="hidden"),
        # mean attention from hidden states: a 48x56 image
        _encode("encode-hidden-mean-48x56", "bf16", 1, 1, 48, 56, 16, 80, 4, 4, 336, 336,
                source="hidden", mean=True),
        # decoder layer of the serving batch: short prompts, half of the visual tokens leave
        _prune("prune-16x192", "bf16", 16, 35, 192, 64, 1, 32, 32, 128, 4096, 96),
        # one long visual span under grouped-query attention
        _prune("prune-gqa-4096", "bf16", 1, 0, 4096, 256, 1, 28, 4, 128, 3584, 2048),
        # large batch, long spans, eight query positions, compacted inside the cache
        _prune("prune-in-place-32x2880", "bf16", 32, 35, 2880, 512, 8, 32, 32, 128, 4096, 288,
               layout="in_place"),
        # dynamic-resolution requests of unequal length in one call
        _prune("prune-ragged-12x1500", "bf16", 12, 40, 1500, 160, 1, 28, 4, 128, 3584, 500,
               layout="ragged", lens_seed=3),
        # stage 2 of a batch scored from hidden states and projection weights
        _prune("prune-hidden-16x576", "bf16", 16, 35, 576, 64, 1, 32, 32, 128, 4096, 192,
               source="hidden"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


#: (heads, head size) of the encoders and (query heads, kv heads, head size, hidden) of the decoders
_ENCODERS = [(16, 64), (12, 64), (16, 80), (8, 64)]
_DECODERS = [(32, 32, 128, 4096), (28, 4, 128, 3584), (16, 16, 64, 1024), (32, 8, 128, 4096)]


def _draw_encode(rng, source, mean):
    dtype = "f32" if rng.random() < 0.25 else "bf16"
    heads, head_dim = rng.choice(_ENCODERS)
    shallow = rng.random() < 0.2
    if mean:
        gh, gw = _log_int(rng, 18, 128), _log_int(rng, 18, 128)
        batch, crops = rng.choice([1, 1, 2, 3]), 1
        # the quadratic part, in units of the largest listed case (fp32 matrix products are an
        # order of magnitude slower; projections from hidden states are scored in fp32)
        slow = 1.0 if dtype == "bf16" and source == "qk" else 12.0
        while batch * (1 + shallow) * slow * (gh * gw) ** 2 * heads * head_dim > 0.9 * 16384 ** 2 * 1280:
            gh, gw = max(9, int(gh * 0.8)), max(9, int(gw * 0.9))
            batch = 1
    else:
        gh, gw = _log_int(rng, 9, 36), _log_int(rng, 9, 36)
        batch, crops = _log_int(rng, 1, 24), rng.choice([1, 1, 1, 2, 5, 8])
        while batch * crops * gh * gw > 24000:
            batch, crops = max(1, batch // 2), max(1, crops - 1)
    n = gh * gw
    wr, wc = rng.randint(1, min(8, gh // 3)), rng.randint(1, min(8, gw // 3))
    kept = max(2, int(n * math.exp(rng.uniform(math.log(0.08), math.log(0.4)))))
    keep_local = min(kept // 2, wr * wc * ((gh // wr) * (gw // wc)))
    c = _encode("", dtype, batch, crops, gh, gw, heads, head_dim, wr, wc, kept - keep_local,
                keep_local, source=source, mean=mean, shallow=shallow,
                all_keys=not mean and rng.random() < 0.25)
    del c["name"]
    return c


def _draw_prune(rng, source, layout):
    dtype = "f32" if rng.random() < 0.2 else "bf16"
    hq, hkv, dh, hidden = rng.choice(_DECODERS)
    n_query = rng.choice([1, 1, 1, 4, 8])
    batch = _log_int(rng, 1, 32)
    prefix, text = rng.randint(0, 80), _log_int(rng, 16, 512)
    vis = _log_int(rng, 48, 4096)
    all_keys = rng.random() < 0.2
    rows = hq // hkv * n_query
    if rows > 64:
        n_query, rows = 1, hq // hkv
    while (vis + (prefix + text if all_keys else 0) + 64) * rows > 34000:
        vis = int(vis * 0.7)
        text = max(16, int(text * 0.7))
    while batch * (prefix + vis + text) > (40000 if dtype == "f32" or source == "hidden" else 90000):
        batch = max(1, batch * 2 // 3)
    keep = max(1, int(vis * rng.uniform(0.05, 0.6)))
    c = _prune("", dtype, batch, prefix, vis, text, n_query, hq, hkv, dh, hidden, keep,
               source=source, layout=layout, all_keys=all_keys, lens_seed=rng.randint(1, 1 << 20))
    del c["name"]
    return c


def draw(rng):
    kind = rng.choices(["cls", "mean", "cls-hidden", "mean-hidden", "dense", "in_place", "ragged",
                        "prune-hidden"], [4, 3, 1, 1, 4, 2, 2, 1])[0]
    if kind in ("cls", "mean"):
        return _draw_encode(rng, "qk", kind == "mean")
    if kind in ("cls-hidden", "mean-hidden"):
        return _draw_encode(rng, "hidden", kind == "mean-hidden")
    if kind == "prune-hidden":
        return _draw_prune(rng, "hidden", "dense")
    return _draw_prune(rng, "qk", kind)


# ------------------------------------------------------------------------------------- shapes
def _encoder_shape(c):
    return wl.EncoderShape(dtype=c["dtype"], batch=c["batch"], n_segments=c["crops"],
                           grid_h=c["grid_h"], grid_w=c["grid_w"], has_cls=0 if c["mean"] else 1,
                           score_mode=vb.VSCAN_SCORE_MEAN_RECEIVED if c["mean"] else vb.VSCAN_SCORE_CLS_ROW,
                           heads=c["heads"], head_dim=c["head_dim"],
                           feat_dim=c["heads"] * c["head_dim"], win_rows=c["win_rows"],
                           win_cols=c["win_cols"], keep_global=c["keep_global"],
                           keep_local=c["keep_local"], softmax_domain=int(c["all_keys"]))


def _llm_shape(c):
    return wl.LlmShape(dtype=c["dtype"], batch=c["batch"], prefix=c["prefix"], vis_len=c["vis"],
                       text=c["text"], n_query=c["n_query"], q_heads=c["q_heads"],
                       kv_heads=c["kv_heads"], head_dim=c["head_dim"], hidden=c["hidden"],
                       keep=c["keep"], in_place=int(c["layout"] == "in_place"),
                       softmax_domain=int(c["all_keys"]))


def _lens(c):
    """(seq_len, vis_start, vis_len, keep) of every sequence; the first one fills the capacities."""
    if c["layout"] != "ragged":
        one = (c["prefix"] + c["vis"] + c["text"], c["prefix"], c["vis"], c["keep"])
        return [one] * c["batch"]
    rng = random.Random(c["lens_seed"])
    out = []
    for b in range(c["batch"]):
        f = 1.0 if b == 0 else rng.uniform(0.15, 1.0)
        vis = max(1, int(c["vis"] * f))
        prefix = rng.randint(0, c["prefix"])
        text = max(c["n_query"], int(c["text"] * rng.uniform(0.3, 1.0)))
        out.append((prefix + vis + text, prefix, vis, min(vis, max(1, int(c["keep"] * f)))))
    return out


# ------------------------------------------------------------------------------------- inputs
def _features(c, gen, dev):
    """Patch features [B, C, N, D] fp32: 48 cluster centres an image plus noise, four tokens a
    segment three times as long."""
    B, C, N, D = c["batch"], c["crops"], c["grid_h"] * c["grid_w"], c["heads"] * c["head_dim"]
    x = torch.randn((B, C, N, D), generator=gen, device=dev) * 0.1
    for b in range(B):
        centres = torch.randn((48, D), generator=gen, device=dev)
        ids = torch.randint(0, 48, (C * N,), generator=gen, device=dev)
        x[b] += centres[ids].view(C, N, D)
    far = torch.rand((B, C, N), generator=gen, device=dev).topk(min(4, N), dim=-1).indices
    x.scatter_(2, far[..., None].expand(-1, -1, -1, D), 3.0 * x.gather(2, far[..., None].expand(-1, -1, -1, D)))
    return x


def _prepare_encode(c, seed):
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(seed)
    shape, dt = _encoder_shape(c), _TORCH[c["dtype"]]
    B, C, S, H, dh, D = (c["batch"], c["crops"], shape.rows, c["heads"], c["head_dim"],
                         shape.feat_dim)
    x = _features(c, gen, dev)
    # logits of a trained encoder spread over a few units: with every token a query the literal
    # recipe's would spread over tens
    gain = 0.25 if c["mean"] else 1.0
    layers = []
    for layer in range(2 if c["shallow"] else 1):
        rows = x
        if shape.has_cls:
            cls = x.mean(dim=2, keepdim=True)
            cls = cls + 0.1 * torch.randn(cls.shape, generator=gen, device=dev)
            rows = torch.cat([cls, x], dim=2)
        if layer:
            rows = rows + 0.5 * torch.randn(rows.shape, generator=gen, device=dev)
        wq = torch.randn((D, H * dh), generator=gen, device=dev) * (0.125 * gain)
        wk = torch.randn((D, H * dh), generator=gen, device=dev) * 0.125
        if c["source"] == "hidden":
            layers.append((rows.to(dt).contiguous(), wq.t().to(dt).contiguous(),
                           wk.to(dt).contiguous()))
        else:
            flat = rows.reshape(B * C * S, D)
            q, k = (torch.mm(flat, w).view(B, C, S, H, dh).transpose(2, 3).to(dt).contiguous()
                    for w in (wq, wk))
            layers.append((q, k))
    desc = vb.encoder_desc(shape)
    size = vb.encoder_fused_workspace_size if c["source"] == "hidden" else vb.encoder_workspace_size
    ws = torch.empty(size(desc, c["shallow"]), dtype=torch.uint8, device=dev)
    return {"case": c, "shape": shape, "layers": layers, "workspace": ws,
            "x": x.view(B, C * shape.n_tokens, D).to(dt).contiguous()}


def _prepare_prune(c, seed):
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(seed)
    shape, dt = _llm_shape(c), _TORCH[c["dtype"]]
    B, S, Hq, Hkv, dh, Dh, Tq = (c["batch"], shape.seq_len, c["q_heads"], c["kv_heads"],
                                 c["head_dim"], c["hidden"], c["n_query"])

    def normal(*size):
        return torch.randn(size, generator=gen, device=dev, dtype=dt)

    st = {"case": c, "shape": shape, "hidden": normal(B, S, Dh)}
    desc = vb.llm_desc(shape)
    if c["source"] == "hidden":
        st["w_q"] = normal(Hq * dh, Dh) * Dh ** -0.5
        st["w_k_t"] = normal(Dh, Hkv * dh) * Dh ** -0.5
        st["workspace"] = torch.empty(vb.llm_fused_workspace_size(desc), dtype=torch.uint8, device=dev)
        return st
    st["k"], st["v"] = normal(B, Hkv, S, dh), normal(B, Hkv, S, dh)
    # a cache that is compacted in place is pruned again for every later question, so a few
    # questions take turns there
    st["q"] = [normal(B, Hq, Tq, dh) for _ in range(6 if c["layout"] == "in_place" else 1)]
    st["turn"] = 0
    toward = 0.5 * st["q"][0].float().view(B, Hkv, -1, dh).mean(dim=2)
    lens = _lens(c)
    rng = random.Random(seed)
    for b, (_, start, vis, _) in enumerate(lens):
        for pos in rng.sample(range(vis), min(4, vis)):
            st["k"][b, :, start + pos] = (st["k"][b, :, start + pos].float() + toward[b]).to(dt)
    if c["layout"] == "ragged":
        st["lens"] = lens
    else:
        st["workspace"] = torch.empty(vb.llm_workspace_size(desc), dtype=torch.uint8, device=dev)
    return st


def prepare(case, seed):
    torch.cuda.set_device(0)
    return (_prepare_encode if case["path"] == "encode" else _prepare_prune)(case, seed)


# ------------------------------------------------------------------------------------- the pass
def run(state):
    c, shape = state["case"], state["shape"]
    if c["path"] == "encode":
        layers = state["layers"]
        if c["source"] == "hidden":
            r = vb.encoder_reduce_fused(shape, *layers[0], state["x"],
                                        local=layers[1] if c["shallow"] else None, want_assign=True,
                                        want_scores=True, workspace=state["workspace"])
        else:
            r = vb.encoder_reduce(shape, *layers[0], state["x"], *(layers[1] if c["shallow"] else ()),
                                  want_assign=True, want_scores=True, workspace=state["workspace"])
        return {n: r[n] for n in ("kept_idx", "merged", "assign", "scores")}
    if c["source"] == "hidden":
        r = vb.llm_prune_fused(shape, state["hidden"], state["w_q"], state["w_k_t"],
                               want_scores=True, workspace=state["workspace"])
        return {n: r[n] for n in ("kept_idx", "hidden", "scores")}
    q = state["q"][state["turn"] % len(state["q"])]
    state["turn"] += 1
    if c["layout"] == "ragged":
        r = vb.llm_prune_ragged(shape, state["lens"], q, state["k"], state["v"], state["hidden"],
                                want_scores=True)
    else:
        r = vb.llm_prune(shape, q, state["k"], state["v"], state["hidden"], want_scores=True,
                         workspace=state["workspace"])
    return {n: r[n] for n in ("kept_idx", "k", "v", "hidden", "scores")}


# ------------------------------------------------------------------------------------- the work
def _work_encode(c):
    es = 2 if c["dtype"] == "bf16" else 4
    shape = _encoder_shape(c)
    B, C, S, N, H, dh, D = (c["batch"], c["crops"], shape.rows, shape.n_tokens, c["heads"],
                            c["head_dim"], shape.feat_dim)
    T, K, BC, layers = shape.tokens_per_image, shape.keep, c["batch"] * c["crops"], 1 + c["shallow"]
    # x in; merged, kept, assignment and scores out; assignment of the dropped to the kept, means
    nbytes = B * (T * D * es + K * D * es + 4 * K + 8 * T)
    flops = B * (2.0 * (T - K) * K * D + T * D)
    if c["source"] == "hidden":
        nbytes += layers * (BC * S * D * es + 2 * D * H * dh * es)
        if c["mean"]:
            flops += layers * BC * (4.0 * S * D * H * dh + 2.0 * H * N * N * dh)
        else:  # one query: it is carried through both projections instead of projecting all keys
            flops += layers * BC * (4.0 * D * H * dh + 2.0 * H * N * D)
    elif c["mean"]:
        nbytes += layers * 2 * BC * H * S * dh * es
        flops += layers * BC * 2.0 * H * N * N * dh
    else:
        nbytes += layers * BC * H * (S + 1) * dh * es
        flops += layers * BC * 2.0 * H * S * dh
    return {"bytes": nbytes, "flops": flops}


def _work_prune(c):
    es = 2 if c["dtype"] == "bf16" else 4
    Hq, Hkv, dh, Dh, Tq = c["q_heads"], c["kv_heads"], c["head_dim"], c["hidden"], c["n_query"]
    nbytes, flops = 0, 0.0
    for seq, start, vis, keep in _lens(c):
        domain = seq if c["all_keys"] else vis
        out = seq - vis + keep
        # rows that have to be copied: in place the ones before the span stay where they are
        moved = out - (start if c["layout"] == "in_place" else 0)
        if c["source"] == "hidden":
            # the domain's hidden states are read once for scores and copies alike
            nbytes += (domain + (0 if c["all_keys"] else moved - keep) + moved) * Dh * es
            flops += 4.0 * Tq * Hq * dh * Dh + 2.0 * domain * Hq * Tq * Dh
        else:
            nbytes += (domain + (0 if c["all_keys"] else moved - keep)) * Hkv * dh * es  # K in
            nbytes += moved * (Hkv * dh + Dh) * es                               # V, hidden in
            nbytes += moved * (2 * Hkv * dh + Dh) * es                           # out
            nbytes += Hq * Tq * dh * es
            flops += 2.0 * domain * Hq * Tq * dh
        nbytes += 4 * (vis + keep)
    if c["source"] == "hidden":
        nbytes += (Hq + Hkv) * dh * Dh * es
    return {"bytes": nbytes, "flops": flops}


def work(case):
    return _work_encode(case) if case["path"] == "encode" else _work_prune(case)


# ------------------------------------------------------------------------------------- tolerance
def tolerance(case):
    # Measured against the definitions in 64 bits.  Prune: the scores are 32-bit sums (at most 4e-7
    # off in the norm, 9e-7 at one value), everything else is copied.  Encode: the same scores
    # (2e-6), but up to 5 tokens in 10^4 have two equally similar kept tokens within 32 bits and
    # join either; a group of one or two members then has another mean (1.6e-3 in fp32, 3e-3 in
    # bf16 in the norm, 0.26 at one value).
    if case["path"] == "prune":
        return {"rel": 5e-6, "max": 1e-5, "differ": 0.01}
    return {"rel": 1e-2 if case["dtype"] == "bf16" else 6e-3, "max": 0.9, "differ": 0.01}
