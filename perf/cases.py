"""The work whose speed is kept an eye on: calls that a user of this library makes, over their real range.

A case is a dict of plain values.  Three kinds:

  block      one transformer block over one packed mini-batch.  op "fwd" is the forward (frozen or
             evaluated block), "step" forward then backward (a training step's share of one layer),
             "recompute" the backward alone with OB_BWD_RECOMPUTE and OB_BWD_ACCUMULATE (a layer whose
             activations were not kept, in a second micro-batch).
  attn       varlen attention alone, forward then backward.
  connector  the ViT -> LLM hand-over, "fwd" or "step".

Segment layouts: "tiles" = image tiles of 1025 tokens; "samples" = LLM samples, 256 visual tokens per
tile plus log-normal text (median 300); "text" = text-only samples; "one" = a single segment.
"""
import math
import random
import types

import numpy as np
import torch

import paper_2407_20761_amd as ob

DEV = "cuda"
TILE = 1025          # 32 x 32 patches and the class token of a 448-pixel tile
PER_TILE = 256       # visual tokens of a tile on the LLM side
TILE_PMF = (0.22, 0.20, 0.16, 0.14, 0.07, 0.06, 0.04, 0.03, 0.03, 0.02, 0.015, 0.015)

# hidden, query heads, kv heads, head size, mlp, layernorm?, swiglu?, causal?, rotary?, biases?, eps
SHAPES = {
    "tiny": (256, 4, 4, 64, 1024, 1, 0, 1, 0, 1, 1e-5),
    "vit-300m": (1024, 16, 16, 64, 4096, 1, 0, 0, 0, 1, 1e-5),
    "llm-7b": (4096, 32, 8, 128, 14336, 0, 1, 1, 1, 0, 1e-6),
    "vit-6b": (3200, 25, 25, 128, 12800, 0, 0, 0, 0, 0, 1e-6),
    "llm-20b": (6144, 48, 8, 128, 16384, 0, 1, 1, 1, 0, 1e-6),
    # sizes off the configurations, as in the tests: a small GQA language model, a ViT of hidden 640
    "llm-small": (768, 12, 4, 64, 2112, 0, 1, 1, 1, 0, 1e-6),
    "vit-small": (640, 10, 10, 64, 2560, 1, 0, 0, 0, 1, 1e-5),
}
MAX_TOKENS = {"tiny": 16384, "vit-300m": 12 * TILE, "llm-7b": 16384, "vit-6b": 16 * TILE, "llm-20b": 32768,
              "llm-small": 16384, "vit-small": 12 * TILE}
CONNECTORS = {"vit-300m": (1024, 4096), "vit-6b": (3200, 6144)}


def _block(name, shape, op, layout, tokens, lens_seed=0):
    return {"name": name, "kind": "block", "shape": shape, "op": op, "layout": layout, "tokens": tokens, "lens_seed": lens_seed}


def _attn(name, nq, nkv, d, causal, layout, tokens, lens_seed=0):
    return {"name": name, "kind": "attn", "nq": nq, "nkv": nkv, "d": d, "causal": causal, "layout": layout, "tokens": tokens,
            "lens_seed": lens_seed}


def _conn(name, shape, op, tiles, lens_seed=0):
    return {"name": name, "kind": "connector", "shape": shape, "op": op, "tiles": tiles, "lens_seed": lens_seed}


def listed():
    return [
        # the smallest block: bring-up and unit-sized training, bound by launches
        _block("tiny-step", "tiny", "step", "samples", 964, 1),
        # one 448-pixel image through a layer of the 300M vision tower
        _block("vit300m-fwd-1tile", "vit-300m", "fwd", "tiles", 1 * TILE),
        # the balanced mini-batch of the 300M vision tower in training
        _block("vit300m-step-12tiles", "vit-300m", "step", "tiles", 12 * TILE),
        # one short sample (a tile and a question) through a layer of the 7B language model
        _block("llm7b-fwd-short", "llm-7b", "fwd", "one", 557),
        # the balanced mini-batch of the 7B language model in training: the headline stack's layer
        _block("llm7b-step-16k", "llm-7b", "step", "samples", 16327, 2),
        # the balanced mini-batch of the 6B vision tower in training
        _block("vit6b-step-16tiles", "vit-6b", "step", "tiles", 16 * TILE),
        # the 6B vision tower under re-computation on a small micro-batch, gradients accumulated
        _block("vit6b-recompute-3tiles", "vit-6b", "recompute", "tiles", 3 * TILE),
        # the balanced mini-batch of the 20B language model in training: the largest call
        _block("llm20b-step-32k", "llm-20b", "step", "samples", 32741, 3),
        # one sample of the greatest length (12 tiles and 4096 tokens of text), 7B heads
        _attn("attn-long-sample", 32, 8, 128, True, "one", 12 * PER_TILE + 4096),
        # text-only samples, many and short, small heads
        _attn("attn-short-texts", 16, 4, 64, True, "text", 8187, 4),
        # hand-over of a 300M vision tower's mini-batch to the 7B model
        _conn("connector-300m-12tiles", "vit-300m", "step", 12, 5),
        # hand-over of the 6B vision tower's mini-batch to the 20B model, the tiles of 16K LLM tokens
        _conn("connector-6b-42tiles", "vit-6b", "step", 42, 6),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    seed = rng.randrange(1 << 20)
    kind = rng.choice(("block", "block", "block", "attn", "connector"))
    if kind == "block":
        shape = rng.choice(sorted(SHAPES))
        op = rng.choice(("fwd", "step", "step", "recompute"))
        if shape.startswith("vit"):
            c = _block("", shape, op, "tiles", TILE * rng.randint(1, MAX_TOKENS[shape] // TILE))
        else:
            c = _block("", shape, op, rng.choice(("samples", "samples", "text", "one")), _log_int(rng, 64, MAX_TOKENS[shape]), seed)
            if c["layout"] == "one":
                c["tokens"] = min(c["tokens"], 12 * PER_TILE + 4096)
    elif kind == "attn":
        d = rng.choice((64, 128))
        nkv = rng.choice((1, 2, 4, 8, 16) if d == 64 else (1, 2, 4, 8))
        nq = nkv * rng.choice((1, 2, 4, 6) if nkv <= 8 else (1, 2))
        causal = rng.random() < 0.6
        layout = rng.choice(("samples", "text", "one")) if causal else "tiles"
        tokens = _log_int(rng, 64, 16384 if layout != "one" else 12 * PER_TILE + 4096) if causal else TILE * rng.randint(1, 16)
        c = _attn("", nq, nkv, d, causal, layout, tokens, seed)
    else:
        c = _conn("", rng.choice(sorted(CONNECTORS)), rng.choice(("fwd", "step")), _log_int(rng, 1, 42), seed)
    del c["name"]
    return c


# ---- segment layouts ---------------------------------------------------------------------------

def _text(rng):
    return max(1, min(4096, int(round(math.exp(math.log(300.0) + rng.gauss(0.0, 1.0))))))


def _lens(case):
    T = case["tokens"]
    if case["layout"] == "tiles":
        return [TILE] * (T // TILE)
    if case["layout"] == "one":
        return [T]
    rng = random.Random(case["lens_seed"])
    lens, total = [], 0
    while total < T:
        n = _text(rng)
        if case["layout"] == "samples":
            n += PER_TILE * rng.choices(range(1, 13), TILE_PMF)[0]
        n = min(n, T - total)
        lens.append(n)
        total += n
    return lens


def _cu(case):
    return np.concatenate([[0], np.cumsum(_lens(case))]).astype(np.int32)


def _visual_rows(case):
    """Rows of the packed LLM batch that hold visual tokens, and the batch's token count: samples of a few
    tiles each, their visual tokens followed by their text."""
    rng = random.Random(case["lens_seed"])
    left, pos, rows = case["tiles"], 0, []
    while left:
        n = min(left, rng.choices(range(1, 13), TILE_PMF)[0])
        rows.append(np.arange(pos, pos + n * PER_TILE, dtype=np.int32))
        pos += n * PER_TILE + _text(rng)
        left -= n
    return np.concatenate(rows), pos


# ---- shapes and inputs -------------------------------------------------------------------------

def _shape(name):
    H, nq, nkv, d, F, ln, glu, causal, rot, bias, eps = SHAPES[name]
    return types.SimpleNamespace(hidden=H, n_q_heads=nq, n_kv_heads=nkv, head_dim=d, mlp_dim=F,
                                 norm=ob.OB_LAYERNORM if ln else ob.OB_RMSNORM, mlp=ob.OB_SWIGLU if glu else ob.OB_GELU,
                                 mask=ob.OB_MASK_SEG_CAUSAL if causal else ob.OB_MASK_SEG_BIDIR, use_rotary=bool(rot),
                                 has_bias=bool(bias), rotary_base=10000.0, norm_eps=eps,
                                 d_qkv=(nq + 2 * nkv) * d, up_rows=F * (2 if glu else 1))


def _weight_shapes(s):
    H = s.hidden
    out = {"n1_g": (H,), "w_qkv": (s.d_qkv, H), "w_o": (H, s.n_q_heads * s.head_dim), "n2_g": (H,), "w_up": (s.up_rows, H),
           "w_down": (H, s.mlp_dim)}
    if s.has_bias:
        out.update({"b_qkv": (s.d_qkv,), "b_o": (H,), "b_up": (s.up_rows,), "b_down": (H,)})
        if s.norm == ob.OB_LAYERNORM:
            out.update({"n1_b": (H,), "n2_b": (H,)})
    return out


def _connector_shapes(Hv, Ht):
    W = 4 * Hv
    return {"n_g": (W,), "n_b": (W,), "w1": (Ht, W), "b1": (Ht,), "w2": (Ht, Ht), "b2": (Ht,)}


def _randn(gen, shape, std=1.0):
    t = torch.randn(shape, generator=gen, device=DEV, dtype=torch.bfloat16)
    return t if std == 1.0 else t.mul_(std)


def _weights(gen, shapes):
    w = {}
    for n in sorted(shapes):
        w[n] = _randn(gen, shapes[n], 0.02)
        if n in ("n1_g", "n2_g", "n_g"):
            w[n] += 1.0
    return w


def _inputs(case, seed):
    """The tensors of a case, from the seed alone: bf16, the order of the draws is part of the case."""
    gen = torch.Generator(device=DEV).manual_seed(int(seed))
    if case["kind"] == "block":
        s = _shape(case["shape"])
        T, H = case["tokens"], s.hidden
        i = {"w": _weights(gen, _weight_shapes(s)), "x": _randn(gen, (T, H), 0.02)}
        if case["op"] != "fwd":
            i["dy"] = _randn(gen, (T, H))
        if case["op"] == "recompute":      # what an earlier micro-batch left
            i["g"] = {n: _randn(gen, t.shape) for n, t in sorted(i["w"].items())}
        return i
    if case["kind"] == "attn":
        T, nq, nkv, d = case["tokens"], case["nq"], case["nkv"], case["d"]
        return {"qkv": _randn(gen, (T, (nq + 2 * nkv) * d)), "d_o": _randn(gen, (T, nq * d))}
    Hv, Ht = CONNECTORS[case["shape"]]
    i = {"w": _weights(gen, _connector_shapes(Hv, Ht)), "v": _randn(gen, (case["tiles"] * TILE, Hv))}
    llm_tokens = _visual_rows(case)[1]
    i["x_llm"] = _randn(gen, (llm_tokens, Ht), 0.02)        # the text rows, already embedded
    if case["op"] != "fwd":
        i["dx_llm"] = _randn(gen, (llm_tokens, Ht))
    return i


def _bytes(n):
    return torch.empty(max(int(n), 256), dtype=torch.uint8, device=DEV)


def prepare(case, seed):
    i = _inputs(case, seed)
    s = {"case": case, **i}
    if case["kind"] == "block":
        T = case["tokens"]
        s["desc"] = ob.make_desc(_shape(case["shape"]))
        s["seg"] = ob.Segments(_cu(case), device=DEV)
        s["saved"] = _bytes(ob.ob_block_saved_bytes(s["desc"], T))
        s["ws"] = _bytes(ob.ob_block_workspace_bytes(s["desc"], T))
        if case["op"] != "recompute":
            s["y"] = torch.empty_like(i["x"])
        if case["op"] != "fwd":
            s["dx"] = torch.empty_like(i["x"])
        if case["op"] == "step":
            s["g"] = {n: torch.empty_like(t) for n, t in i["w"].items()}
    elif case["kind"] == "attn":
        T, nq, nkv, d = case["tokens"], case["nq"], case["nkv"], case["d"]
        s["seg"] = ob.Segments(_cu(case), device=DEV)
        s["o"], s["lse"] = torch.empty_like(i["d_o"]), torch.empty((nq, T), dtype=torch.float32, device=DEV)
        s["dqkv"] = torch.empty_like(i["qkv"])
        s["ws"] = _bytes(ob.ob_varlen_attn_bwd_workspace_bytes(T, nq, nkv, d))
    else:
        Hv, Ht = CONNECTORS[case["shape"]]
        rows, s["llm_tokens"] = _visual_rows(case)
        s["rows"] = ob.RowIndex(rows, device=DEV)
        s["desc"] = ob.make_connector_desc(Hv, Ht, 32, 1e-5)
        s["saved"] = _bytes(ob.ob_connector_saved_bytes(s["desc"], case["tiles"]))
        s["ws"] = _bytes(ob.ob_connector_workspace_bytes(s["desc"], case["tiles"]))
        if case["op"] != "fwd":
            s["dv"] = torch.empty_like(i["v"])
            s["g"] = {n: torch.empty_like(t) for n, t in i["w"].items()}
    return s


def run(s):
    case = s["case"]
    if case["kind"] == "block":
        if case["op"] == "recompute":
            ob.ob_block_bwd(s["desc"], s["w"], s["g"], ob.OB_BWD_ACCUMULATE | ob.OB_BWD_RECOMPUTE, s["x"], s["dy"], s["dx"],
                            s["saved"], s["seg"], s["ws"])
            return {"dx": s["dx"], "g": s["g"]}
        ob.ob_block_fwd(s["desc"], s["w"], s["x"], s["y"], s["saved"], s["seg"], s["ws"])
        if case["op"] == "fwd":
            return {"y": s["y"]}
        ob.ob_block_bwd(s["desc"], s["w"], s["g"], 0, s["x"], s["dy"], s["dx"], s["saved"], s["seg"], s["ws"])
        return {"y": s["y"], "dx": s["dx"], "g": s["g"]}
    if case["kind"] == "attn":
        nq, nkv, d = case["nq"], case["nkv"], case["d"]
        mask = ob.OB_MASK_SEG_CAUSAL if case["causal"] else ob.OB_MASK_SEG_BIDIR
        qkv, dqkv, ld = s["qkv"], s["dqkv"], s["qkv"].shape[1]
        q, k, v = qkv[:, :nq * d], qkv[:, nq * d:(nq + nkv) * d], qkv[:, (nq + nkv) * d:]
        dq, dk, dv = dqkv[:, :nq * d], dqkv[:, nq * d:(nq + nkv) * d], dqkv[:, (nq + nkv) * d:]
        ob.ob_varlen_attn_fwd(q, k, v, s["o"], s["lse"], ld, ld, nq * d, s["seg"], nq, nkv, d, d ** -0.5, mask)
        ob.ob_varlen_attn_bwd(s["d_o"], q, k, v, s["o"], s["lse"], dq, dk, dv, ld, ld, nq * d, s["seg"], nq, nkv, d,
                              d ** -0.5, mask, s["ws"])
        return {"o": s["o"], "lse": s["lse"], "dq": dq, "dk": dk, "dv": dv}
    ob.ob_connector_fwd(s["desc"], s["w"], s["v"], case["tiles"], s["rows"], s["x_llm"], s["llm_tokens"], s["saved"], s["ws"])
    if case["op"] == "fwd":
        return {"x_llm": s["x_llm"]}
    ob.ob_connector_bwd(s["desc"], s["w"], s["g"], 0, s["v"], s["dx_llm"], s["dv"], case["tiles"], s["rows"], s["llm_tokens"],
                        s["saved"], s["ws"])
    return {"x_llm": s["x_llm"], "dv": s["dv"], "g": s["g"]}


# ---- work, tolerance ---------------------------------------------------------------------------

def _numel(shapes):
    return sum(int(np.prod(v)) for v in shapes.values())


def _area(lens, causal):
    return float(sum(n * (n + 1) // 2 if causal else n * n for n in lens))


def work(case):
    if case["kind"] == "block":
        s = _shape(case["shape"])
        T, H = case["tokens"], s.hidden
        params, act = 2.0 * _numel(_weight_shapes(s)), 2.0 * T * H
        HD = s.n_q_heads * s.head_dim
        attn = 4.0 * HD * _area(_lens(case), s.mask == ob.OB_MASK_SEG_CAUSAL)
        up = 2.0 * T * H * (s.d_qkv + HD + s.up_rows)
        down = 2.0 * T * H * s.mlp_dim
        if case["op"] == "fwd":
            return {"bytes": params + 2 * act, "flops": up + down + attn}
        if case["op"] == "step":      # x, dy, y, dx; weights in, gradients out
            return {"bytes": 2 * params + 4 * act, "flops": 3 * (up + down + attn)}
        # x, dy, dx; weights in, gradients in and out; the replay needs no down projection
        return {"bytes": 3 * params + 3 * act, "flops": 3 * (up + attn) + 2 * down}
    if case["kind"] == "attn":
        T, nq, nkv, d = case["tokens"], case["nq"], case["nkv"], case["d"]
        # q, k, v, d_o in; o, dq, dk, dv and the log-sum-exp out
        return {"bytes": 2.0 * T * d * (4 * nq + 4 * nkv) + 4.0 * nq * T,
                "flops": 3 * 4.0 * nq * d * _area(_lens(case), case["causal"])}
    Hv, Ht = CONNECTORS[case["shape"]]
    n_tok = case["tiles"] * PER_TILE
    params, v, z = 2.0 * _numel(_connector_shapes(Hv, Ht)), 2.0 * case["tiles"] * TILE * Hv, 2.0 * n_tok * Ht
    flops = 2.0 * n_tok * (4 * Hv * Ht + Ht * Ht)
    if case["op"] == "fwd":
        return {"bytes": params + v + z, "flops": flops}
    return {"bytes": 2 * params + 2 * v + 2 * z, "flops": 3 * flops}


def tolerance(case):
    """Measured against exact(): LayerNorm blocks are 0.0015 - 0.0057 off, RMSNorm blocks (residual stream of 0.02,
    a SwiGLU or a wide MLP behind it) 0.0066 - 0.015, attention 0.002 - 0.003, the connector 0.0017 - 0.0039: bf16
    roundings of every stored intermediate.  About four times that; a block's at most 0.03."""
    if case["kind"] == "attn":
        return {"rel": 0.012, "max": 0.25}
    if case["kind"] == "connector":
        return {"rel": 0.016, "max": 0.25}
    return {"rel": 0.022 if case["shape"] in ("tiny", "vit-300m", "vit-small") else 0.03, "max": 0.5}


# ---- the same in 64 bits -----------------------------------------------------------------------

def _norm(x, g, b, eps, layer):
    """(normalised rows times gain plus offset, the saved values of the backward)"""
    mu = x.mean(1, keepdim=True) if layer else torch.zeros_like(x[:, :1])
    c = x - mu
    r = (c.square().mean(1, keepdim=True) + eps).rsqrt()
    n = c * r
    return n * g + (0 if b is None else b), (n, r)


def _norm_bwd(dy, g, saved, layer):
    n, r = saved
    dn = dy * g
    d = dn - n * (dn * n).mean(1, keepdim=True)
    if layer:
        d = d - dn.mean(1, keepdim=True)
    return d * r, (dy * n).sum(0), dy.sum(0)


def _gelu(x):
    return 0.5 * x * (1 + torch.erf(x / math.sqrt(2)))


def _gelu_d(x):
    return 0.5 * (1 + torch.erf(x / math.sqrt(2))) + x * torch.exp(-0.5 * x * x) / math.sqrt(2 * math.pi)


def _heads(lens, nq, nkv, d):
    at = 0
    for n in lens:
        for a in range(nq):
            b = a // (nq // nkv)
            yield slice(at, at + n), slice(a * d, (a + 1) * d), slice(b * d, (b + 1) * d), a
        at += n


def _scores(q, k, causal, scale):
    S = (q @ k.t()) * scale
    if causal:
        n = S.shape[0]
        S.masked_fill_(torch.ones((n, n), dtype=torch.bool, device=S.device).triu_(1), -math.inf)
    return S


def _attn_fwd(q, k, v, lens, nq, nkv, d, causal, scale):
    o = torch.empty_like(q)
    lse = torch.empty((nq, q.shape[0]), dtype=torch.float64, device=q.device)
    for t, cq, ck, a in _heads(lens, nq, nkv, d):
        S = _scores(q[t, cq], k[t, ck], causal, scale)
        lse[a, t] = torch.logsumexp(S, 1)
        o[t, cq] = torch.exp(S - lse[a, t][:, None]) @ v[t, ck]
    return o, lse


def _attn_bwd(do, q, k, v, o, lse, lens, nq, nkv, d, causal, scale):
    dq, dk, dv = torch.empty_like(q), torch.zeros_like(k), torch.zeros_like(v)
    for t, cq, ck, a in _heads(lens, nq, nkv, d):
        P = torch.exp(_scores(q[t, cq], k[t, ck], causal, scale) - lse[a, t][:, None])
        dv[t, ck] += P.t() @ do[t, cq]
        delta = (do[t, cq] * o[t, cq]).sum(1, keepdim=True)
        dS = P * (do[t, cq] @ v[t, ck].t() - delta) * scale
        dq[t, cq] = dS @ k[t, ck]
        dk[t, ck] += dS.t() @ q[t, cq]
    return dq, dk, dv


def _rotate(x, pos, d, sign):
    half = d // 2
    freq = 10000.0 ** (-2.0 * torch.arange(half, dtype=torch.float64, device=x.device) / d)
    ang = pos[:, None] * freq[None, :]
    c, s = torch.cos(ang)[:, None, :], sign * torch.sin(ang)[:, None, :]
    y = x.view(x.shape[0], -1, d)
    lo, hi = y[..., :half], y[..., half:]
    return torch.cat([lo * c - hi * s, hi * c + lo * s], -1).reshape(x.shape)


def _exact_block(case, i):
    s = _shape(case["shape"])
    lens = _lens(case)
    w = {n: t.double() for n, t in i["w"].items()}
    x = i["x"].double()
    nq, nkv, d, F = s.n_q_heads, s.n_kv_heads, s.head_dim, s.mlp_dim
    layer, causal, scale = s.norm == ob.OB_LAYERNORM, s.mask == ob.OB_MASK_SEG_CAUSAL, s.head_dim ** -0.5
    b = lambda n: w.get(n, 0)  # noqa: E731
    pos = torch.cat([torch.arange(n, device=DEV) for n in lens]).double()
    Q, K = nq * d, (nq + nkv) * d
    h1, sv1 = _norm(x, w["n1_g"], w.get("n1_b"), s.norm_eps, layer)
    qkv = h1 @ w["w_qkv"].t() + b("b_qkv")
    q, k, v = qkv[:, :Q], qkv[:, Q:K], qkv[:, K:]
    if s.use_rotary:
        q, k = _rotate(q, pos, d, 1.0), _rotate(k, pos, d, 1.0)
    o, lse = _attn_fwd(q, k, v, lens, nq, nkv, d, causal, scale)
    x1 = x + o @ w["w_o"].t() + b("b_o")
    h2, sv2 = _norm(x1, w["n2_g"], w.get("n2_b"), s.norm_eps, layer)
    up = h2 @ w["w_up"].t() + b("b_up")
    if s.mlp == ob.OB_SWIGLU:
        act = up[:, :F] * torch.sigmoid(up[:, :F]) * up[:, F:]
    else:
        act = _gelu(up)
    y = x1 + act @ w["w_down"].t() + b("b_down") if case["op"] != "recompute" else None
    if case["op"] == "fwd":
        return {"y": y}
    dy = i["dy"].double()
    g = {"w_down": dy.t() @ act, "b_down": dy.sum(0)}
    dact = dy @ w["w_down"]
    if s.mlp == ob.OB_SWIGLU:
        gate, lin = up[:, :F], up[:, F:]
        sg = torch.sigmoid(gate)
        dup = torch.cat([dact * lin * sg * (1 + gate * (1 - sg)), dact * gate * sg], 1)
    else:
        dup = dact * _gelu_d(up)
    del dact, act, up
    g["w_up"], g["b_up"] = dup.t() @ h2, dup.sum(0)
    dh, g["n2_g"], g["n2_b"] = _norm_bwd(dup @ w["w_up"], w["n2_g"], sv2, layer)
    del dup
    dx1 = dy + dh
    g["w_o"], g["b_o"] = dx1.t() @ o, dx1.sum(0)
    dq, dk, dv = _attn_bwd(dx1 @ w["w_o"], q, k, v, o, lse, lens, nq, nkv, d, causal, scale)
    if s.use_rotary:
        dq, dk = _rotate(dq, pos, d, -1.0), _rotate(dk, pos, d, -1.0)
    dqkv = torch.cat([dq, dk, dv], 1)
    g["w_qkv"], g["b_qkv"] = dqkv.t() @ h1, dqkv.sum(0)
    dh, g["n1_g"], g["n1_b"] = _norm_bwd(dqkv @ w["w_qkv"], w["n1_g"], sv1, layer)
    g = {n: g[n] for n in i["w"]}
    if case["op"] == "recompute":
        return {"dx": dx1 + dh, "g": {n: g[n] + i["g"][n].double() for n in g}}
    return {"y": y, "dx": dx1 + dh, "g": g}


def _exact_attn(case, i):
    nq, nkv, d = case["nq"], case["nkv"], case["d"]
    lens, scale = _lens(case), case["d"] ** -0.5
    qkv, do = i["qkv"].double(), i["d_o"].double()
    q, k, v = qkv[:, :nq * d].contiguous(), qkv[:, nq * d:(nq + nkv) * d].contiguous(), qkv[:, (nq + nkv) * d:].contiguous()
    o, lse = _attn_fwd(q, k, v, lens, nq, nkv, d, case["causal"], scale)
    dq, dk, dv = _attn_bwd(do, q, k, v, o, lse, lens, nq, nkv, d, case["causal"], scale)
    return {"o": o, "lse": lse, "dq": dq, "dk": dk, "dv": dv}


def _patch_rows(tiles):
    """[tokens, 4] rows of v that make up each sub-sampled token: 2 x 2 patches, row-major."""
    t, r, c = torch.meshgrid(torch.arange(tiles), torch.arange(16), torch.arange(16), indexing="ij")
    at = [t * TILE + 1 + (2 * r + dr) * 32 + 2 * c + dc for dr in (0, 1) for dc in (0, 1)]
    return torch.stack([a.reshape(-1) for a in at], 1).to(DEV)


def _exact_connector(case, i):
    w = {n: t.double() for n, t in i["w"].items()}
    rows = torch.from_numpy(_visual_rows(case)[0]).to(DEV).long()
    v = i["v"].double()
    src = _patch_rows(case["tiles"])
    u = v[src].reshape(src.shape[0], -1)
    un, sv = _norm(u, w["n_g"], w["n_b"], 1e-5, True)
    h = un @ w["w1"].t() + w["b1"]
    a = _gelu(h)
    x = i["x_llm"].double()
    x[rows] = a @ w["w2"].t() + w["b2"]
    if case["op"] == "fwd":
        return {"x_llm": x}
    dz = i["dx_llm"].double()[rows]
    g = {"w2": dz.t() @ a, "b2": dz.sum(0)}
    dh = (dz @ w["w2"]) * _gelu_d(h)
    g["w1"], g["b1"] = dh.t() @ un, dh.sum(0)
    du, g["n_g"], g["n_b"] = _norm_bwd(dh @ w["w1"], w["n_g"], sv, True)
    dv = torch.zeros_like(v)
    dv[src.reshape(-1)] = du.reshape(-1, v.shape[1])
    return {"x_llm": x, "dv": dv, "g": g}


def exact(case, seed):
    i = _inputs(case, seed)
    return {"block": _exact_block, "attn": _exact_attn, "connector": _exact_connector}[case["kind"]](case, i)
