"""The work that programs have this library do, as cases that can be timed.

A case is a dict of plain values.  Four kinds:

- ``block``: one ``foe.cluster_block`` call (the whole MoE block of C co-resident
  clusters), at the sizes of decode steps, of small and medium batches and of
  prefill chunks;
- ``steps``: the block from its single steps for a program with a router of its
  own: per cluster ``foe.permute``, ``foe.expert_ffn`` and ``foe.combine``, then
  ``foe.reduce``;
- ``route``: ``foe.route`` alone, for a program that only needs the decisions;
- ``attn``: one ``foe.group_attention`` call over one sequence.

Every state keeps its workspace and output buffers, as a serving loop does.
Activations are N(0, 1) and weights N(0, sigma) with sigma near 1/sqrt(d), the
scales that the library's synthetic workloads use.
"""

from __future__ import annotations

import math

import torch

from paper_2605_06206_amd import foe

# Rotary base and position scaling of both attention models.
THETA, ROPE_SCALE = 500000.0, 16.0


def listed():
    block = dict(kind="block", dtype="bf16", gating="renorm", zipf=0.0)
    return [
        # One token through the eight clusters of a layer that share the GPU
        # (the 7B share): a decode step of a single request.
        dict(block, name="decode_one", C=8, T=1, d=2048, E=8, k=2, F=1024),
        # A decode step of 128 requests through one cluster.
        dict(block, name="decode_batch", C=1, T=128, d=2048, E=16, k=2, F=1024),
        # A medium batch (many requests decoding, or one short prompt): about
        # 64 rows per expert, between the decode and the prefill sizes.
        dict(block, name="mid_batch", C=1, T=512, d=2048, E=16, k=2, F=1024),
        # A prompt whose length and widths fit no tile, with the globally
        # normalised gating and a router bias.
        dict(block, name="ragged_global", C=2, T=777, d=1000, E=12, k=3, F=680,
             gating="global", zipf=0.5),
        # The prefill-shaped block with a Zipf(1.2) skewed router.
        dict(block, name="prefill_zipf", C=1, T=8192, d=2048, E=16, k=2, F=1024, zipf=1.2),
        # All eight clusters of a 7B layer on one GPU over a 4096-token chunk.
        dict(block, name="layer_share", C=8, T=4096, d=2048, E=8, k=2, F=1024),
        # The largest block: wide model, many experts, four slots per token.
        dict(block, name="large", C=1, T=16384, d=4096, E=32, k=4, F=1536),
        # 32-bit weights and activations: a small model evaluated in full
        # precision.
        dict(block, name="block_fp32", dtype="f32", C=1, T=384, d=768, E=8, k=2, F=512),
        # The single steps, two clusters, a router of the program's own.
        dict(kind="steps", name="steps", dtype="bf16", C=2, T=2048, d=2048, E=16, k=2, F=1024,
             skew=0.5),
        # A short prompt through the 1B model's attention (one query head per
        # group, head size 96).
        dict(kind="attn", name="attn_1b_short", H=8, S=1000, d=768, nq=1, hd=96),
        # A 4096-token prefill chunk through the 7B model's attention (two
        # query heads per group, head size 128).
        dict(kind="attn", name="attn_7b", H=8, S=4096, d=2048, nq=2, hd=128),
        # The longest sequence: the attention product itself dominates.
        dict(kind="attn", name="attn_7b_long", H=8, S=32768, d=2048, nq=2, hd=128),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi):
    """A row width: mostly multiples of 128, else any multiple of 8."""
    step = 128 if rng.random() < 0.6 else 8
    return max(step, _log_int(rng, lo, hi) // step * step)


def draw(rng):
    """One more case of the ranges above."""
    what = rng.choice(["decode", "decode", "mid", "mid", "prefill", "prefill", "ragged", "fp32",
                       "steps", "route", "attn", "attn"])
    if what == "attn":
        big = rng.random() < 0.5
        S = _log_int(rng, 64, 16384) + rng.choice([0, 0, 1, 7])
        return dict(kind="attn", H=rng.choice([4, 8, 8]), S=S, d=2048 if big else 768,
                    nq=rng.choice([2, 2, 1, 4]) if big else rng.choice([1, 1, 2]),
                    hd=128 if big else 96)
    if what == "steps":
        return dict(kind="steps", dtype="bf16",
                    C=rng.choice([1, 2, 4]), T=_log_int(rng, 16, 1024), d=_width(rng, 512, 2048),
                    E=rng.choice([8, 12, 16]), k=rng.choice([1, 2, 4]), F=_width(rng, 256, 1024),
                    skew=rng.choice([0.0, 0.5, 1.2]))
    if what == "route":
        return dict(kind="route", dtype="bf16", gating=rng.choice(["renorm", "global"]),
                    C=rng.choice([1, 4, 8]), T=_log_int(rng, 1, 16384), d=_width(rng, 768, 4096),
                    E=rng.choice([8, 16, 32]), k=rng.choice([1, 2, 4]), zipf=rng.choice([0.0, 1.2]))
    c = dict(kind="block", dtype="bf16", gating=rng.choice(["renorm", "renorm", "global"]),
             zipf=rng.choice([0.0, 0.0, 0.5, 1.2]))
    if what == "fp32":
        return dict(c, dtype="f32", C=1, T=_log_int(rng, 16, 384),
                    d=_width(rng, 128, 768), E=rng.choice([4, 8, 12]), k=rng.choice([1, 2]),
                    F=_width(rng, 128, 512))
    if what == "ragged":
        return dict(c, C=rng.choice([1, 2, 3, 4]), T=_log_int(rng, 1, 2000),
                    d=8 * rng.randint(25, 250), E=rng.randint(1, 32), k=1,
                    F=8 * rng.randint(20, 150))
    lo, hi = {"decode": (1, 128), "mid": (128, 2048), "prefill": (2048, 12000)}[what]
    return dict(c, C=rng.choice([1, 1, 2, 4, 8]) if what == "decode" else rng.choice([1, 1, 2, 4]),
                T=_log_int(rng, lo, hi), d=128 * rng.randint(8, 20), E=rng.choice([8, 16, 24, 32]),
                k=rng.choice([1, 2, 2, 4]), F=64 * rng.randint(8, 20))


# ---- inputs ------------------------------------------------------------------


def _dtype(case):
    return torch.float32 if case.get("dtype") == "f32" else torch.bfloat16


def _normal(gen, shape, sigma, dtype):
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).mul_(sigma).to(dtype)


def _weights(gen, case, dtype):
    C, E, d, F = case["C"], case["E"], case["d"], case["F"]
    sigma = 1.0 / math.sqrt(d)
    w = {}
    for name, shape in (("w_gate", (E, F, d)), ("w_up", (E, F, d)), ("w_down", (E, d, F))):
        w[name] = torch.empty((C,) + shape, dtype=dtype, device="cuda")
        for h in range(C):
            w[name][h] = _normal(gen, shape, sigma, dtype)
    return w


def _router(gen, case, dtype):
    C, E, d = case["C"], case["E"], case["d"]
    w = _normal(gen, (C, E, d), 1.0 / math.sqrt(d), dtype)
    bias = None
    if case["zipf"]:
        rank = torch.arange(1, E + 1, dtype=torch.float64, device="cuda")
        bias = (-case["zipf"] * rank.log()).float().repeat(C, 1).contiguous()
    return w, bias


def _inputs(case, seed):
    """The tensors a program holds before the call, from the seed alone."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dtype = _dtype(case)
    kind = case["kind"]
    if kind == "attn":
        H, S, d, nq, hd = (case[n] for n in ("H", "S", "d", "nq", "hd"))
        sigma = 1.0 / math.sqrt(d)
        return {"x": _normal(gen, (H, S, d), 1.0, dtype),
                "w_qkv": _normal(gen, (H, (nq + 2) * hd, d), sigma, dtype),
                "w_o": _normal(gen, (d, H * nq * hd), sigma, dtype)}
    C, T, d, E, k = (case[n] for n in ("C", "T", "d", "E", "k"))
    st = {"x": _normal(gen, (T, d), 1.0, dtype)}
    if kind in ("block", "route"):
        st["w_router"], st["bias"] = _router(gen, case, dtype)
    if kind == "steps":
        # k distinct experts per token, drawn with the skew, and their weights
        u = torch.rand((C, T, E), generator=gen, device="cuda", dtype=torch.float64)
        score = -(-(u.clamp(1e-12, 1 - 1e-12)).log()).log()
        score -= case["skew"] * torch.arange(1, E + 1, device="cuda", dtype=torch.float64).log()
        top, idx = score.topk(k, dim=-1)
        st["topk_idx"] = idx.int().contiguous()
        st["topk_w"] = top.float().softmax(-1).contiguous()
    if kind in ("block", "steps"):
        st.update(_weights(gen, case, dtype))
    return st


def prepare(case, seed):
    st = _inputs(case, seed)
    st["case"] = case
    kind, dt = case["kind"], foe.F32 if case.get("dtype") == "f32" else foe.BF16
    x = st["x"]
    if kind == "attn":
        H, S, d, nq, hd = (case[n] for n in ("H", "S", "d", "nq", "hd"))
        st["out"] = torch.empty((S, d), dtype=x.dtype, device="cuda")
        nbytes = foe.lib().foe_group_attention_workspace_bytes(H, S, d, nq, hd)
        st["ws"] = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        return st
    C, T, d, E, k = (case[n] for n in ("C", "T", "d", "E", "k"))
    if kind == "block":
        nbytes = foe.workspace_bytes("cluster_block", dt, C, T, d, E, k, case["F"])
        st["ws"] = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        st["out"] = torch.empty_like(x)
    elif kind == "route":
        st["topk_idx"] = torch.empty((C, T, k), dtype=torch.int32, device="cuda")
        st["topk_w"] = torch.empty((C, T, k), dtype=torch.float32, device="cuda")
    else:
        nbytes = max(foe.workspace_bytes("permute", dt, 1, T, d, E, k, 0),
                     foe.workspace_bytes("expert_ffn", dt, 1, T * k, d, E, 1, case["F"]), 1)
        st["ws"] = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        st["y"] = torch.empty((T * k, d), dtype=x.dtype, device="cuda")
        st["partials"] = torch.empty((C, T, d), dtype=x.dtype, device="cuda")
        st["out"] = torch.empty_like(x)
    return st


# ---- one pass ----------------------------------------------------------------


def run(st):
    case, kind = st["case"], st["case"]["kind"]
    if kind == "attn":
        return foe.group_attention(st["x"], st["w_qkv"], st["w_o"], case["nq"], THETA, ROPE_SCALE,
                                   out=st["out"], ws=st["ws"])
    if kind == "block":
        return foe.cluster_block(st["x"], st["w_router"], st["bias"], st["w_gate"], st["w_up"],
                                 st["w_down"], case["k"], out=st["out"], ws=st["ws"],
                                 gating=case["gating"])
    if kind == "route":
        return foe.route(st["x"], st["w_router"], st["bias"], case["k"], st["topk_idx"],
                         st["topk_w"], gating=case["gating"])
    outs = []
    for h in range(case["C"]):
        p = foe.permute(st["topk_idx"][h], st["x"], case["E"], ws=st["ws"])
        foe.expert_ffn(p["x_perm"], p["offsets"], st["w_gate"][h], st["w_up"][h], st["w_down"][h],
                       y_perm=st["y"], ws=st["ws"])
        foe.combine(st["y"], p["row_of"], st["topk_w"][h], out=st["partials"][h])
        outs.append(p)
    foe.reduce(st["partials"], 1.0 / case["C"], residual=st["x"], out=st["out"])
    return {"dispatch": outs, "partials": st["partials"], "out": st["out"]}


# ---- what a pass cannot do without -----------------------------------------------


def work(case):
    el = 4 if case.get("dtype") == "f32" else 2
    if case["kind"] == "attn":
        H, S, d, nq, hd = (case[n] for n in ("H", "S", "d", "nq", "hd"))
        proj = 2 * H * S * d * (nq + 2) * hd + 2 * S * d * H * nq * hd
        core = 4 * hd * nq * H * S * (S + 1) // 2
        return {"bytes": el * (H * S * d + H * (nq + 2) * hd * d + d * H * nq * hd + S * d),
                "flops": proj + core}
    C, T, d, E, k = (case[n] for n in ("C", "T", "d", "E", "k"))
    route = {"bytes": el * (T * d + C * E * d) + 8 * C * T * k, "flops": 2 * C * T * d * E}
    if case["kind"] == "route":
        return route
    F = case["F"]
    hit = E * (1.0 - (1.0 - k / E) ** T)  # experts of a cluster that receive rows, uniform routing
    weights = int(C * hit * 3 * F * d * el)
    flops = 6 * C * T * k * d * F
    if case["kind"] == "block":
        return {"bytes": weights + el * (2 * T * d + C * E * d), "flops": flops + route["flops"]}
    rows = C * T * k
    return {"bytes": weights + el * (2 * T * d + rows * d + C * T * d) + 16 * rows, "flops": flops}


def tolerance(case):
    """About four times the error against 64 bits: one rounding of the output to bf16 leaves
    1.7e-3 (2.9e-3 where the residual is not part of it), 32-bit sums 3e-7."""
    if case["kind"] == "route":
        # the weights are 32-bit; a near tie of two scores may pick another expert
        return {"rel": 2e-6, "differ": 1e-3}
    if case.get("dtype") == "f32":
        return {"rel": 2e-6, "differ": 0.0}
    return {"rel": 1.2e-2 if case["kind"] == "steps" else 7e-3, "differ": 0.0}


# ---- the same in 64 bits ---------------------------------------------------------


def _select(scores, k, gating):
    """Top-k of [T, C, E] scores per cluster (equal scores: lower id) and weights."""
    order = torch.sort(scores, dim=-1, descending=True, stable=True)
    idx, top = order.indices[..., :k], order.values[..., :k]
    if gating == "global":
        z = torch.logsumexp(scores.flatten(1), dim=1)
        w = (top - z[:, None, None]).exp()
    else:
        w = top.softmax(-1)
    return idx.transpose(0, 1), w.transpose(0, 1)  # [C, T, k]


def _moe(x, idx, w, w_gate, w_up, w_down):
    """sum_j w[:, j] FFN_{idx[:, j]}(x) of one cluster."""
    out = torch.zeros_like(x)
    for e in range(w_gate.shape[0]):
        tok, slot = (idx == e).nonzero(as_tuple=True)
        if tok.numel() == 0:
            continue
        xe = x[tok]
        g, u = xe @ w_gate[e].double().t(), xe @ w_up[e].double().t()
        y = (g * torch.sigmoid(g) * u) @ w_down[e].double().t()
        out.index_add_(0, tok, y * w[tok, slot][:, None])
    return out


def _attention(st, case):
    H, S, d, nq, hd = (case[n] for n in ("H", "S", "d", "nq", "hd"))
    half = hd // 2
    inv = THETA ** (-2.0 * torch.arange(half, dtype=torch.float64, device="cuda") / hd)
    ang = (torch.arange(S, dtype=torch.float64, device="cuda") / ROPE_SCALE)[:, None] * inv
    cos, sin = ang.cos(), ang.sin()

    def rotate(v):
        a, b = v[:, :half], v[:, half:]
        return torch.cat([a * cos - b * sin, b * cos + a * sin], dim=1)

    total = torch.zeros((S, d), dtype=torch.float64, device="cuda")
    keys = torch.arange(S, device="cuda")
    step = max(64, (1 << 25) // S)
    for h in range(H):
        x = st["x"][h].double()
        total += x
        qkv = x @ st["w_qkv"][h].double().t()
        kk, v = rotate(qkv[:, nq * hd:(nq + 1) * hd]), qkv[:, (nq + 1) * hd:]
        for i in range(nq):
            q = rotate(qkv[:, i * hd:(i + 1) * hd]) / math.sqrt(hd)
            o = torch.empty((S, hd), dtype=torch.float64, device="cuda")
            for a in range(0, S, step):
                b = min(a + step, S)
                s = q[a:b] @ kk[:b].t()
                s.masked_fill_(keys[None, :b] > keys[a:b, None], -math.inf)
                o[a:b] = s.softmax(-1) @ v[:b]
            col = (h * nq + i) * hd
            total += o @ st["w_o"][:, col:col + hd].double().t()
    return total / H


def exact(case, seed):
    st = _inputs(case, seed)
    if case["kind"] == "attn":
        return _attention(st, case)
    C, T, E, k = (case[n] for n in ("C", "T", "E", "k"))
    x = st["x"].double()
    if case["kind"] in ("block", "route"):
        scores = torch.einsum("td,ced->tce", x, st["w_router"].double())
        if st["bias"] is not None:
            scores = scores + st["bias"].double()
        idx, w = _select(scores, k, case["gating"])
        if case["kind"] == "route":
            return (None, w)
    else:
        idx, w = st["topk_idx"].long(), st["topk_w"].double()
    parts = [_moe(x, idx[h], w[h], st["w_gate"][h], st["w_up"][h], st["w_down"][h])
             for h in range(C)]
    out = x + sum(parts) / C
    if case["kind"] == "block":
        return out
    dispatch = []
    for h in range(C):
        order = torch.argsort(idx[h].reshape(-1), stable=True)
        dispatch.append({"counts": None, "offsets": None, "sorted_src": None, "row_of": None,
                         "x_perm": x[order // k]})
    return {"dispatch": dispatch, "partials": torch.stack(parts), "out": out}
