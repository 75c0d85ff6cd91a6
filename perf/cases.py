"""The workloads that this library's speed is judged by.

A case is a dict of plain values: `op` (the entry point), the sizes
B, H, L, d, the band half-width w, and for `plan` and `module` the plan code.
Every case is one call of a public entry point of the Python binding, as a
program that samples from a diffusion transformer issues it per layer and
denoising step:

  plan     dfa_plan_step: the attention of one layer at one step under a code
  qkv, out dfa_qkv_proj, dfa_out_proj: the projections around it
  module   dfa_module_step: projection, attention and projection in one call
  mrae     dfa_mrae: the loss of the plan search between two outputs

The listed sizes are the repository's own workloads: `inputs.CONFIGS` (H = 16,
d = 72, w = L / 8; DiT-XL/2 at 256 and 512 px, PixArt-Sigma at 1024 and
2048 px, the spatial and temporal attention of Open-Sora at 240p with 16
frames, and the tiny WA-RS check at d = 64).  `draw` spreads over the same
ranges: 2 to 16384 tokens, ragged lengths, other head counts, both head dims,
all codes that compute.

Q, K, V and hidden states are N(0, 1) rounded to bf16 (inputs.device_qkv);
weights N(0, 1/C).  The residual that a reuse step adds is drawn directly, in
fp32, at the size a refresh leaves (the mean of N(0, 1) values over the band).
"""
from __future__ import annotations

import math

import torch

from paper_2406_08552_amd import dfa, inputs

CODES = {"full": dfa.FULL, "refresh": dfa.WARS_REFRESH, "reuse": dfa.WARS_REUSE, "asc": dfa.ASC_REUSE,
         "asc_refresh": dfa.WARS_ASC_REFRESH, "asc_reuse": dfa.WARS_ASC_REUSE}
HALF = ("asc", "asc_refresh", "asc_reuse")       # computed on the conditional half of the batch
REFRESH, REUSE = ("refresh", "asc_refresh"), ("reuse", "asc_reuse")
DEVICE = "cuda"


def _workload(name, config, op, code=None):
    c = inputs.CONFIGS[config]
    case = {"name": name, "op": op, "B": c.B, "H": c.H, "L": c.L, "d": c.d, "w": c.w}
    if code:
        case["code"] = code
    return case


def listed():
    return [
        # the smallest call: one layer of the tiny d = 64 check, where launch and host latency count
        _workload("tiny_refresh", "tiny", "plan", "refresh"),
        # a reuse step of a small image model: a short band walk, residual read in fp32
        _workload("dit256_reuse", "dit256", "plan", "reuse"),
        # the output projection of that model: few tokens, a small grid
        _workload("dit256_out", "dit256", "out"),
        # video: thousands of 16-token sequences across frames
        _workload("temporal_reuse", "opensora_temporal", "plan", "reuse"),
        # video: 405-token sequences within frames (ragged tiles); the step that makes the residual
        _workload("spatial_refresh", "opensora_spatial", "plan", "refresh"),
        # a whole uncompressed module of a 512 px image model: both projections and attention
        _workload("dit512_module", "dit512", "module", "full"),
        # 1024 px: the conditional half computed and stored to both halves
        _workload("pixart1k_asc", "pixart1k", "plan", "asc"),
        # 1024 px: the step that makes the residual, at an ordinary length
        _workload("pixart1k_refresh", "pixart1k", "plan", "refresh"),
        # 2048 px, the largest: full attention, the band-only step, and the QKV projection
        _workload("pixart2k_full", "pixart2k", "plan", "full"),
        _workload("pixart2k_reuse", "pixart2k", "plan", "reuse"),
        _workload("pixart2k_qkv", "pixart2k", "qkv"),
        # the plan search's loss between two 2048 px module outputs
        _workload("pixart2k_mrae", "pixart2k", "mrae"),
    ]


MAX_ELEMS = 2 * 16 * 16384 * 72                    # elements of one tensor of the largest listed case
MAX_PAIRS = 2 * 16 * 16384 * 16384                 # its (query, key) pairs


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["plan"] * 6 + ["short", "qkv", "out", "module", "module", "mrae"])
    d = rng.choice([72, 72, 64])
    if op == "short":                              # many short sequences
        L = rng.randint(2, 32)
        B, H = 2 * _log_int(rng, 16, 512), rng.choice([8, 12, 16])
        w = rng.randint(1, max(1, L // 4))
        return {"op": "plan", "code": rng.choice(["full", "refresh", "reuse", "asc"]), "B": B, "H": H, "L": L, "d": d, "w": w}
    L = _log_int(rng, 33, 16384)
    B = 2 * _log_int(rng, 1, 16)
    if op in ("qkv", "out", "module"):             # C = H * d is a multiple of 128
        H = rng.choice([16, 16, 32]) if d == 72 else rng.choice([6, 8, 12, 16, 24])
    else:
        H = rng.choice([16, 16, 16, 2, 6, 8, 12, 24])
    elems = MAX_ELEMS // 2 if op == "module" else MAX_ELEMS
    pairs = MAX_PAIRS // 2 if op in ("plan", "module") else None
    while B > 2 and (B * H * L * d > elems or (pairs and B * H * L * L > pairs)):
        B = max(2, (B // 4) * 2)
    while B * H * L * d > elems or (pairs and B * H * L * L > pairs):
        L = max(33, L * 3 // 4)
    w = rng.choice([max(1, L // 8)] * 3 + [rng.randint(1, max(1, L // 4))])
    case = {"op": op, "B": B, "H": H, "L": L, "d": d, "w": w}
    if op == "plan":
        case["code"] = rng.choice(["full", "refresh", "refresh", "reuse", "reuse", "asc", "asc_refresh", "asc_reuse"])
    elif op == "module":
        case["code"] = rng.choice(["full", "refresh", "reuse", "asc"])
    return case


def _band(L, w):
    """(query, key) pairs of one sequence inside |i - j| <= w."""
    return L * L if w >= L - 1 else L * (2 * w + 1) - w * (w + 1)


def _randn(g, shape, scale=1.0, dtype=torch.bfloat16):
    return (torch.randn(shape, generator=g, device=DEVICE, dtype=torch.float32) * scale).to(dtype)


def prepare(case, seed):
    op, code = case["op"], case.get("code")
    B, H, L, d, w = (case[k] for k in ("B", "H", "L", "d", "w"))
    C = H * d
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    s = {"op": op, "code": code, "w": w, "H": H, "B": B}
    heads, tokens = (B, H, L, d), (B, L, C)
    if op == "mrae":
        s["A"] = _randn(g, tokens)
        s["other"] = (s["A"].float() + _randn(g, tokens, 0.05, torch.float32)).to(torch.bfloat16)
        s["workspace"] = torch.empty(dfa.MRAE_WORKSPACE_BYTES, dtype=torch.uint8, device=DEVICE)
        s["result"] = torch.empty(1, dtype=torch.float64, device=DEVICE)
        return s
    if op in ("qkv", "module"):
        s["X"] = _randn(g, tokens)
        s["Wqkv"] = _randn(g, (3 * C, C), C ** -0.5)
        s["bqkv"] = _randn(g, (3 * C,), 0.1, torch.float32)
    if op in ("out", "module"):
        s["Wo"] = _randn(g, (C, C), C ** -0.5)
        s["bo"] = _randn(g, (C,), 0.1, torch.float32)
        s["Y"] = torch.empty(tokens, dtype=torch.bfloat16, device=DEVICE)
    for name in ("Q", "K", "V"):
        if op == "plan":
            s[name] = _randn(g, heads)
        elif op != "out":
            s[name] = torch.empty(heads, dtype=torch.bfloat16, device=DEVICE)
    if op == "out":
        s["O"] = _randn(g, heads)
    elif op != "qkv":
        s["O"] = torch.empty(heads, dtype=torch.bfloat16, device=DEVICE)
    if code in REUSE:
        s["R"] = _randn(g, heads, (2 * w + 1) ** -0.5, torch.float32)
    elif code in REFRESH:
        s["R"] = torch.empty(heads, dtype=torch.float32, device=DEVICE)
    return s


def run(s):
    op, code = s["op"], s["code"]
    if op == "mrae":
        dfa.dfa_mrae(s["A"], s["other"], s["workspace"], s["result"])
        return s["result"]
    if op == "qkv":
        dfa.dfa_qkv_proj(s["X"], s["Wqkv"], s["bqkv"], s["Q"], s["K"], s["V"])
        return {"Q": s["Q"], "K": s["K"], "V": s["V"]}
    if op == "out":
        dfa.dfa_out_proj(s["O"], s["Wo"], s["bo"], s["Y"])
        return s["Y"]
    R = s.get("R")
    if op == "plan":
        dfa.dfa_plan_step(CODES[code], s["Q"], s["K"], s["V"], s["O"], R, s["O"], s["w"])
        out = {"O": s["O"]}
    else:
        dfa.dfa_module_step(CODES[code], s["X"], s["Wqkv"], s["bqkv"], s["Wo"], s["bo"], s["Q"], s["K"], s["V"], s["O"],
                            R, s["Y"], s["Y"], s["w"], s["H"])
        out = {"Y": s["Y"]}
    if code in REFRESH:   # the combined codes write the conditional half alone
        out["R"] = R[: s["B"] // 2] if code in HALF else R
    return out


def work(case):
    op, code = case["op"], case.get("code")
    B, H, L, d, w = (case[k] for k in ("B", "H", "L", "d", "w"))
    C, n = H * d, B * H * L * d
    if op == "mrae":
        return {"bytes": 4 * n + 8, "flops": 6 * n}
    if op == "qkv":
        return {"bytes": 2 * n + 6 * C * C + 12 * C + 6 * n, "flops": 6 * n * C}
    if op == "out":
        return {"bytes": 2 * n + 2 * C * C + 4 * C + 2 * n, "flops": 2 * n * C}
    half = 0.5 if code in HALF else 1
    pairs = B * H * (_band(L, w) if code in REUSE else L * L) * half
    residual = 4 * n * half if code in REFRESH + REUSE else 0
    if op == "plan":
        return {"bytes": 6 * n * half + 2 * n + residual, "flops": 4 * d * pairs}
    return {"bytes": 2 * n * half + 2 * n + 8 * C * C + 16 * C + residual, "flops": 4 * d * pairs + 8 * n * C * half}


def tolerance(case):
    # About four times the error of the outputs against 64 bits, measured on
    # the listed cases and drawn ones: bf16 outputs of bf16 probabilities.
    op = case["op"]
    if op == "mrae":
        return {"rel": 1e-6}                       # fp32 lane sums added in fp64: 4e-9 seen, another order up to 1e-7
    if op in ("qkv", "out"):
        return {"rel": 7e-3, "max": 1.6e-2}        # one rounding to bf16: 1.7e-3 and 3.9e-3 seen
    if op == "plan":
        return {"rel": 1e-2, "max": 6e-2}          # 2.3e-3 and 1.5e-2 seen
    return {"rel": 1.4e-2, "max": 6.5e-2}          # bf16 between the three stages: 3.4e-3 and 1.6e-2 seen


def _attention64(Q, K, V, w=None):
    """softmax(Q K^T / sqrt(d)) V of [N, L, d] fp64 tensors (inside the band where w is given)."""
    N, L, d = Q.shape
    out = torch.empty_like(Q)
    rows = min(L, max(1, (1 << 27) // L))
    heads = max(1, (1 << 27) // (rows * L))
    j = torch.arange(L, device=Q.device)
    for n0 in range(0, N, heads):
        kt = K[n0:n0 + heads].transpose(1, 2).contiguous()
        v = V[n0:n0 + heads]
        for i0 in range(0, L, rows):
            S = torch.matmul(Q[n0:n0 + heads, i0:i0 + rows], kt) * d ** -0.5
            if w is not None:
                i = torch.arange(i0, min(L, i0 + rows), device=Q.device)
                S.masked_fill_((i[:, None] - j[None, :]).abs() > w, float("-inf"))
            out[n0:n0 + heads, i0:i0 + rows] = torch.matmul(torch.softmax(S, dim=-1), v)
    return out


def _attend64(code, Q, K, V, R, w):
    """The outputs of one plan code, [B, H, L, d] fp64: O, and R of a refresh."""
    B, H, L, d = Q.shape
    P = B // 2 if code in HALF else B
    q, k, v = (t[:P].reshape(P * H, L, d) for t in (Q, K, V))
    win = _attention64(q, k, v, w).view(P, H, L, d) if code in REFRESH + REUSE else None
    if code in REUSE:
        o = win + R[:P].double()
    else:
        o = _attention64(q, k, v).view(P, H, L, d)
    res = o - win if code in REFRESH else None
    return (torch.cat([o, o]) if code in HALF else o), res


def exact(case, seed):
    s = prepare(case, seed)
    op, code = case["op"], case.get("code")
    B, H, L, d, w = (case[k] for k in ("B", "H", "L", "d", "w"))
    C = H * d
    if op == "mrae":
        a, b = s["A"].double(), s["other"].double()
        e = (a - b).abs() / (torch.maximum(a.abs(), b.abs()) + 1e-6)
        return e.clamp_(0, 10).mean().reshape(1)
    if op in ("qkv", "module"):
        qkv = torch.matmul(s["X"].double(), s["Wqkv"].double().t().contiguous()) + s["bqkv"].double()
        Q, K, V = qkv.view(B, L, 3, H, d).permute(2, 0, 3, 1, 4).contiguous()
        if op == "qkv":
            return {"Q": Q, "K": K, "V": V}
    if op == "out":
        O = s["O"].double()
    else:
        if op == "plan":
            Q, K, V = (s[n].double() for n in ("Q", "K", "V"))
        O, res = _attend64(code, Q, K, V, s.get("R"), w)
    if op == "plan":
        out = {"O": O}
    else:
        merged = O.permute(0, 2, 1, 3).reshape(B, L, C)
        Y = torch.matmul(merged, s["Wo"].double().t().contiguous()) + s["bo"].double()
        if op == "out":
            return Y
        out = {"Y": Y}
    if code in REFRESH:
        out["R"] = res
    return out
