"""The calls whose speed on one MI355X is followed: what a program that decodes with a 4-bit target model asks of this
library, each through its public entry points (paper_2505_22179_amd/binding.py) on device buffers that such a program
keeps -- packed weights, caches, workspaces.  Shapes are the Llama-3 8B / 70B layer shapes of inputs.py and generic
ones with ragged sizes; token counts are those of plain decoding (1), sequence verification (about 7), draft beams
(about 10) and tree verification (24 .. 64)."""
from __future__ import annotations

import math

import torch

from paper_2505_22179_amd import binding as B
from paper_2505_22179_amd import inputs as I

DEV = "cuda"
G = 128
D = 128          # head dimension of every attention here
EPS = 1e-5
MODELS = {       # hidden, query heads, KV heads, feed-forward width
    "8b": (4096, 32, 8, 14336),
    "70b": (8192, 64, 8, 28672),
}
MAX_WEIGHTS = 57344 * 8192   # the largest linear of the 70B layer


def listed():
    return [
        # plain decoding: one token through one square projection, the smallest call of a decode step
        {"name": "linear_m1_4096x4096", "kind": "linear", "M": 1, "K": 4096, "N": 4096, "epi": "none", "sym": False},
        # plain decoding: the widest linear of a 70B layer with its SiLU gate
        {"name": "linear_m1_70b_gate_up", "kind": "linear", "M": 1, "K": 8192, "N": 57344, "epi": "silu", "sym": False},
        # verification of a sequence draft: the longest contraction, residual added, symmetrically quantised weight
        {"name": "linear_m7_70b_down_sym", "kind": "linear", "M": 7, "K": 28672, "N": 8192, "epi": "residual", "sym": True},
        # tree verification on the 8B intermediate model: q/k/v projection with rotary embedding and cache append
        {"name": "rope_m30_8b_qkv", "kind": "rope", "M": 30, "K": 4096, "Hq": 32, "Hkv": 8, "P": 2048},
        # tree verification on a model of another size: a shape no launch table knows, columns not a multiple of 128
        {"name": "linear_m37_ragged", "kind": "linear", "M": 37, "K": 5120, "N": 13000, "epi": "none", "sym": False},
        # tree verification of 60 nodes: the widest linear of a 70B layer with its gate
        {"name": "linear_m60_70b_gate_up", "kind": "linear", "M": 60, "K": 8192, "N": 57344, "epi": "silu", "sym": False},
        # tree attention of the 70B verification step
        {"name": "attn_m60_70b_p2048", "kind": "attn", "M": 60, "P": 2048, "Hq": 64, "Hkv": 8},
        # tree attention of the 8B model behind a long document
        {"name": "attn_m40_8b_p16001", "kind": "attn", "M": 40, "P": 16001, "Hq": 32, "Hkv": 8},
        # plain decoding: one whole layer of the 8B model
        {"name": "layer_m1_8b", "kind": "layer", "M": 1, "P": 2048, "hidden": 4096, "Hq": 32, "Hkv": 8, "ffn": 14336, "sym": False},
        # tree verification: one whole layer of the 70B model
        {"name": "layer_m60_70b", "kind": "layer", "M": 60, "P": 2048, "hidden": 8192, "Hq": 64, "Hkv": 8, "ffn": 28672, "sym": False},
        # one step of a beam-search draft: language-model head, log-softmax and the ten best tokens of ten beams
        {"name": "lm_head_m10_8b", "kind": "lm_head", "M": 10, "K": 4096, "V": 128256, "top_k": 10},
        # the verifying model's own head: greedy token of every tree node
        {"name": "lm_head_m60_70b", "kind": "lm_head", "M": 60, "K": 8192, "V": 128256, "top_k": 1},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["linear", "linear", "linear", "rope", "attn", "attn", "layer", "lm_head"])
    M = _log_int(rng, 1, 64) if rng.random() < 0.5 else rng.randint(1, 64)
    if kind == "linear":
        if rng.random() < 0.4:
            _, K, N = rng.choice(I.LLAMA3_8B + I.LLAMA3_70B)
        else:
            K = 128 * _log_int(rng, 8, 224)
            N = 32 * _log_int(rng, 32, min(1792, MAX_WEIGHTS // K // 32))
        epi = rng.choice(["none", "residual", "silu"])
        if epi != "silu" and rng.random() < 0.5:
            N -= 8 * rng.randint(0, 3)   # ragged column counts
        return {"kind": "linear", "M": M, "K": K, "N": N, "epi": epi, "sym": rng.random() < 0.3}
    heads = rng.choice([(32, 8), (64, 8), (40, 8), (16, 2), (12, 2), (8, 8)])
    if kind == "rope":
        return {"kind": "rope", "M": M, "K": 128 * _log_int(rng, 8, 64), "Hq": heads[0], "Hkv": heads[1], "P": _log_int(rng, 16, 8192)}
    if kind == "attn":
        return {"kind": "attn", "M": M, "P": _log_int(rng, 16, 20000), "Hq": heads[0], "Hkv": heads[1]}
    if kind == "layer":
        if rng.random() < 0.5:
            hidden, Hq, Hkv, ffn = rng.choice([MODELS["8b"], MODELS["70b"]])
        else:
            Hq, Hkv = heads
            hidden, ffn = Hq * D, 128 * rng.randint(2 * Hq, 4 * Hq)
        return {"kind": "layer", "M": M, "P": _log_int(rng, 16, 8192), "hidden": hidden, "Hq": Hq, "Hkv": Hkv, "ffn": ffn,
                "sym": rng.random() < 0.3}
    return {"kind": "lm_head", "M": M, "K": 128 * _log_int(rng, 8, 64), "V": _log_int(rng, 2000, 128256), "top_k": rng.randint(1, 16)}


# ---- inputs: the distributions of inputs.py, drawn on the device --------------------------------------


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _normal(gen, *shape, std=1.0):
    return (torch.randn(*shape, generator=gen, device=DEV) * std).to(torch.float16)


def _weight(gen, K, N, sym):
    """canonical quantised weight: uniform 4-bit codes, scales in [1e-3, 1e-2], zero-points uniform (or all 8)"""
    qw = torch.randint(-2 ** 31, 2 ** 31, (K // 8, N), dtype=torch.int32, generator=gen, device=DEV)
    sc = (torch.rand(K // G, N, generator=gen, device=DEV) * 9e-3 + 1e-3).to(torch.float16)
    if sym:
        qz = torch.full((K // G, N // 8), -2004318072, dtype=torch.int32, device=DEV)   # 0x88888888
    else:
        qz = torch.randint(-2 ** 31, 2 ** 31, (K // G, N // 8), dtype=torch.int32, generator=gen, device=DEV)
    return qw, sc, qz


def _pack(weight, K, N, how="plain"):
    packed = torch.empty(B.w4a16_packed_bytes(N, K), dtype=torch.uint8, device=DEV)
    if how == "heads":
        B.w4a16_pack_heads(*weight, packed, N, K, D)
    else:
        (B.w4a16_pack_gate_up if how == "gate_up" else B.w4a16_pack)(*weight, packed, N, K)
    return packed


def _tree(seed, M, P):
    """ancestor mask and positions of a draft tree of M nodes behind P committed tokens"""
    if M > 8:
        parent, _, mask = I.make_tree(seed, M, 6, 4)
    else:
        parent, _, mask = I.chain_tree(M)
    return torch.from_numpy(mask).to(DEV), torch.from_numpy(I.tree_positions(parent, P)).to(DEV)


def _tables(n_pos):
    cos, sin = I.make_rope_tables(n_pos, D)
    return torch.from_numpy(cos).to(DEV), torch.from_numpy(sin).to(DEV)


def _inputs(case, seed):
    """what the caller's model and data provide, from the seed alone"""
    gen, kind, M = _gen(seed), case["kind"], case["M"]
    s = {}
    if kind == "linear":
        K, N = case["K"], case["N"]
        s["x"] = _normal(gen, M, K)
        s["weight"] = _weight(gen, K, N, case["sym"])
        if case["epi"] == "residual":
            s["residual"] = _normal(gen, M, N)
    elif kind == "rope":
        K, P, Hq, Hkv = case["K"], case["P"], case["Hq"], case["Hkv"]
        s["x"] = _normal(gen, M, K)
        s["weight"] = _weight(gen, K, (Hq + 2 * Hkv) * D, False)
        s["k"], s["v"] = _normal(gen, P + M, Hkv, D), _normal(gen, P + M, Hkv, D)
        _, s["pos"] = _tree(seed, M, P)
        s["cos"], s["sin"] = _tables(P + 64)
    elif kind == "attn":
        P, Hq, Hkv = case["P"], case["Hq"], case["Hkv"]
        s["q"] = _normal(gen, M, Hq, D)
        s["k"], s["v"] = _normal(gen, P + M, Hkv, D), _normal(gen, P + M, Hkv, D)
        s["mask"], _ = _tree(seed, M, P)
    elif kind == "layer":
        H, Hq, Hkv, F, P = case["hidden"], case["Hq"], case["Hkv"], case["ffn"], case["P"]
        s["h"] = _normal(gen, M, H)
        s["g1"], s["g2"] = 1 + _normal(gen, H, std=0.1), 1 + _normal(gen, H, std=0.1)
        s["qkv"] = _weight(gen, H, (Hq + 2 * Hkv) * D, case["sym"])
        s["o"] = _weight(gen, Hq * D, H, case["sym"])
        s["gate_up"] = _weight(gen, H, 2 * F, case["sym"])
        s["down"] = _weight(gen, F, H, case["sym"])
        s["k"], s["v"] = _normal(gen, P + M, Hkv, D), _normal(gen, P + M, Hkv, D)
        s["mask"], s["pos"] = _tree(seed, M, P)
        s["cos"], s["sin"] = _tables(P + 64)
    else:
        s["x"] = _normal(gen, M, case["K"])
        s["W"] = _normal(gen, case["V"], case["K"], std=0.02)
    return s


def prepare(case, seed):
    s, kind, M = _inputs(case, seed), case["kind"], case["M"]
    s["case"] = case
    half = lambda *shape: torch.empty(*shape, dtype=torch.float16, device=DEV)
    if kind == "linear":
        K, N = case["K"], case["N"]
        s["packed"] = _pack(s.pop("weight"), K, N, "gate_up" if case["epi"] == "silu" else "plain")
        s["y"] = half(M, N // 2 if case["epi"] == "silu" else N)
        s["ws"] = B.new_workspace(B.w4a16_workspace_bytes(M, N, K))
    elif kind == "rope":
        K, N = case["K"], (case["Hq"] + 2 * case["Hkv"]) * D
        s["packed"] = _pack(s.pop("weight"), K, N, "heads")
        s["q"] = half(M, case["Hq"], D)
        s["ws"] = B.new_workspace(B.w4a16_workspace_bytes(M, N, K))
    elif kind == "attn":
        s["out"] = half(M, case["Hq"], D)
        s["ws"] = B.new_workspace(B.tree_verify_attn_workspace_bytes(M, case["P"], case["Hq"], case["Hkv"], D))
    elif kind == "layer":
        H, Hq, Hkv, F, P = case["hidden"], case["Hq"], case["Hkv"], case["ffn"], case["P"]
        Nqkv = (Hq + 2 * Hkv) * D
        shapes = ((Nqkv, H), (H, Hq * D), (2 * F, H), (H, F))
        s["packed"] = (_pack(s.pop("qkv"), H, Nqkv, "heads"), _pack(s.pop("o"), Hq * D, H),
                       _pack(s.pop("gate_up"), H, 2 * F, "gate_up"), _pack(s.pop("down"), F, H))
        s["scratch"] = (half(M, H), None, half(M, Hq, D), half(M, Hq, D), half(M, F),
                        B.new_workspace(max(B.w4a16_workspace_bytes(M, N, K) for N, K in shapes)),
                        B.new_workspace(B.tree_verify_attn_workspace_bytes(M, P, Hq, Hkv, D)))
        s["lw"] = B.layer_weights(*s["packed"], s["g1"], s["g2"], H, Hq, Hkv, D, F, EPS, qkv_heads_packed=True, symmetric=case["sym"])
        s["ls"] = B.layer_scratch(*s["scratch"])
        s["stream_h"] = half(M, H)
    else:
        K, V, k = case["K"], case["V"], case["top_k"]
        s["packed"] = torch.empty(B.lm_head_packed_bytes(V, K), dtype=torch.uint8, device=DEV)
        B.lm_head_pack(s.pop("W"), s["packed"], V, K)
        s["logits"] = torch.empty(M, V, device=DEV)
        s["top_idx"] = torch.empty(M, k, dtype=torch.int32, device=DEV)
        s["top_logprob"] = torch.empty(M, k, device=DEV)
        s["ws"] = torch.empty(B.lm_head_workspace_bytes(M, V, K, k), dtype=torch.uint8, device=DEV)
    return s


def run(s):
    case = s["case"]
    kind, M = case["kind"], case["M"]
    if kind == "linear":
        K, N, epi = case["K"], case["N"], case["epi"]
        if epi == "none" and not case["sym"]:
            B.w4a16_gemm(s["x"], s["packed"], s["y"], M, N, K, G, s["ws"])
        else:
            code = {"none": B.EPI_NONE, "residual": B.EPI_RESIDUAL, "silu": B.EPI_SILU_MUL}[epi] | (B.SYMMETRIC if case["sym"] else 0)
            B.w4a16_gemm_fused(s["x"], s["packed"], s["y"], M, N, K, G, code, s.get("residual"), s["ws"])
        return s["y"]
    if kind == "rope":
        B.w4a16_gemm_rope(s["x"], s["packed"], M, case["K"], G, s["pos"], s["cos"], s["sin"], s["cos"].shape[0], s["q"], s["k"], s["v"],
                          case["P"], case["Hq"], case["Hkv"], D, s["ws"])
        return s["q"], s["k"], s["v"]
    if kind == "attn":
        B.tree_verify_attn(s["q"], s["k"], s["v"], s["mask"], s["out"], M, case["P"], case["Hq"], case["Hkv"], D, D ** -0.5, s["ws"])
        return s["out"]
    if kind == "layer":
        s["stream_h"].copy_(s["h"])   # the hidden state arrives from the layer before
        B.w4a16_decoder_layer(s["lw"], s["stream_h"], M, case["P"], s["pos"], s["cos"], s["sin"], s["cos"].shape[0], s["mask"], s["k"],
                              s["v"], s["ls"])
        return s["stream_h"], s["k"], s["v"]
    B.lm_head_topk(s["x"], s["packed"], M, case["V"], case["K"], case["top_k"], s["logits"], s["top_idx"], s["top_logprob"], s["ws"])
    return s["logits"], s["top_idx"], s["top_logprob"]


def _linear_work(M, K, N, out, sym):
    """codes, scales and (unless the caller vouches for 8) zero-points once, activations once"""
    per_group = 2 * N + (0 if sym else N // 2)
    return K * N // 2 + K // G * per_group + 2 * M * K + 2 * M * out, 2.0 * M * K * N


def _attn_work(M, P, Hq, Hkv):
    return 2 * (2 * M * Hq * D + 2 * (P + M) * Hkv * D) + M * M, 4.0 * M * (P + M) * Hq * D


def work(case):
    kind, M = case["kind"], case["M"]
    if kind == "linear":
        K, N = case["K"], case["N"]
        b, f = _linear_work(M, K, N, N // 2 if case["epi"] == "silu" else N, case["sym"])
        return {"bytes": b + (2 * M * N if case["epi"] == "residual" else 0), "flops": f}
    if kind == "rope":
        N = (case["Hq"] + 2 * case["Hkv"]) * D
        b, f = _linear_work(M, case["K"], N, N, False)
        return {"bytes": b + 4 * M * D, "flops": f}
    if kind == "attn":
        b, f = _attn_work(M, case["P"], case["Hq"], case["Hkv"])
        return {"bytes": b, "flops": f}
    if kind == "layer":
        H, Hq, Hkv, F, sym = case["hidden"], case["Hq"], case["Hkv"], case["ffn"], case["sym"]
        parts = [_linear_work(M, H, (Hq + 2 * Hkv) * D, 0, sym), _linear_work(M, Hq * D, H, 0, sym), _linear_work(M, H, 2 * F, 0, sym),
                 _linear_work(M, F, H, 0, sym)]
        kv = 2 * 2 * (case["P"] + M) * Hkv * D
        return {"bytes": sum(b for b, _ in parts) - 2 * M * (H + Hq * D + H + F) + kv + 4 * M * H + 4 * H,
                "flops": sum(f for _, f in parts) + _attn_work(M, case["P"], Hq, Hkv)[1]}
    K, V, k = case["K"], case["V"], case["top_k"]
    return {"bytes": 2 * V * K + 2 * M * K + 4 * M * V + 8 * M * k, "flops": 2.0 * M * K * V}


def tolerance(case):
    kind = case["kind"]
    # about four times what the results show against 64 bits
    if kind == "linear" or kind == "rope":
        return {"rel": 1e-3}                    # one rounding to fp16 (2.1e-4), rotary outputs two (2.9e-4)
    if kind == "attn":
        return {"rel": 1.1e-3}                  # probabilities and output are rounded to fp16 (2.7e-4)
    if kind == "layer":
        return {"rel": 7e-3}                    # seven fp16 intermediates in a row (7e-4 at M = 1, 1.8e-3 at M = 60)
    return {"rel": 1e-5, "differ": 0.02}        # fp32 sums (6e-7); tokens of nearly equal logits may swap


# ---- the same in 64 bits ------------------------------------------------------------------------------


def _matmul64(x, weight):
    """x [M, K] (fp64) times the dequantised weight, a slice of columns at a time"""
    qw, sc, qz = weight
    K, N = qw.shape[0] * 8, qw.shape[1]
    shifts = torch.arange(0, 32, 4, dtype=torch.int32, device=DEV)
    out = torch.empty(x.shape[0], N, dtype=torch.float64, device=DEV)
    step = max(8, (1 << 27) // K // 8 * 8)
    for n in range(0, N, step):
        e = min(N, n + step)
        q = ((qw[:, None, n:e] >> shifts[None, :, None]) & 15).reshape(K, e - n).double()
        z = ((qz[:, n // 8:e // 8, None] >> shifts) & 15).reshape(K // G, e - n).double()
        w = (q.view(K // G, G, e - n) - z[:, None]) * sc[:, None, n:e].double()
        out[:, n:e] = x @ w.reshape(K, e - n)
    return out


def _attend64(q, k, v, mask, P):
    M, Hq, Hkv = q.shape[0], q.shape[1], k.shape[1]
    out = torch.empty(M, Hq, D, dtype=torch.float64, device=DEV)
    hidden = torch.cat([torch.zeros(M, P, dtype=torch.bool, device=DEV), mask == 0], 1)
    for h in range(Hq):
        g = h // (Hq // Hkv)
        s = (q[:, h] @ k[:, g].t().contiguous()) * D ** -0.5
        out[:, h] = torch.softmax(s.masked_fill(hidden, -math.inf), 1) @ v[:, g].contiguous()
    return out


def _rotate64(x, pos, cos, sin):
    c, s = cos[pos.long()].double()[:, None], sin[pos.long()].double()[:, None]
    a, b = x[..., :D // 2], x[..., D // 2:]
    return torch.cat([a * c - b * s, b * c + a * s], -1)


def _qkv64(n, weight, s, case):
    Hq, Hkv, M, P = case["Hq"], case["Hkv"], case["M"], case["P"]
    qkv = _matmul64(n, weight).view(M, Hq + 2 * Hkv, D)
    q = _rotate64(qkv[:, :Hq], s["pos"], s["cos"], s["sin"])
    k, v = s["k"].double(), s["v"].double()
    k[P:] = _rotate64(qkv[:, Hq:Hq + Hkv], s["pos"], s["cos"], s["sin"])
    v[P:] = qkv[:, Hq + Hkv:]
    return q, k, v


def _silu_mul64(gu):
    g, u = gu.chunk(2, 1)
    return g / (1 + torch.exp(-g)) * u


def _norm64(h, g):
    return h * g.double() / torch.sqrt((h * h).mean(1, keepdim=True) + EPS)


def exact(case, seed):
    s, kind = _inputs(case, seed), case["kind"]
    if kind == "linear":
        y = _matmul64(s["x"].double(), s["weight"])
        return _silu_mul64(y) if case["epi"] == "silu" else y + s["residual"].double() if case["epi"] == "residual" else y
    if kind == "rope":
        return _qkv64(s["x"].double(), s["weight"], s, case)
    if kind == "attn":
        return _attend64(s["q"].double(), s["k"].double(), s["v"].double(), s["mask"], case["P"])
    if kind == "layer":
        h = s["h"].double()
        q, k, v = _qkv64(_norm64(h, s["g1"]), s["qkv"], s, case)
        a = _attend64(q, k, v, s["mask"], case["P"])
        h = h + _matmul64(a.reshape(case["M"], -1), s["o"])
        h = h + _matmul64(_silu_mul64(_matmul64(_norm64(h, s["g2"]), s["gate_up"])), s["down"])
        return h, k, v
    logits = torch.empty(case["M"], case["V"], dtype=torch.float64, device=DEV)
    x = s["x"].double()
    for n in range(0, case["V"], 16384):
        logits[:, n:n + 16384] = x @ s["W"][n:n + 16384].double().t().contiguous()
    top = torch.topk(torch.log_softmax(logits, 1), case["top_k"], 1).values
    return logits, None, top   # tokens of nearly equal logits have no value of their own
