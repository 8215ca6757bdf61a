"""The library's workloads: what its users have it do, with sizes, inputs, cost and expected accuracy.

A case is a dict of plain values.  `listed()` gives the named ones, `draw()` more of the same ranges,
`prepare()` what a program holds before the call (weights, activations, caches, workspace), `run()` one pass
through the public entry points, `work()` the bytes and operations a pass cannot do without, `exact()` the same
outputs in 64 bits from plain torch, `tolerance()` how far a correct fp16 implementation may be from another.

Kinds of pass:
  layer      RMSNorm-QKV, O projection and SwiGLU MLP of one decoder layer, one after the other
  step       one whole decode step of a layer: RMSNorm-QKV with rotary embedding, the new keys and values into the
             caches, attention, O projection + residual, RMSNorm + MLP + residual
  qkv        RMSNorm-QKV with rotary embedding
  linear     a plain projection;  residual: the same with the residual added behind
  norm_mlp   RMSNorm + SwiGLU MLP + residual;  mlp: the SwiGLU MLP alone
  attention  decode attention over per-request caches of unequal lengths
"""
from __future__ import annotations

import math

import torch

import paper_2605_25655_amd as thi

EPS = 1e-6

# hidden, stacked QKV rows, columns of it that are rotated (Q and K), MLP width, head size, weight spread
SHAPES = {
    "tiny": dict(H=512, N=1536, rot=1024, I=1376, hd=64, sigma=0.02),
    "7b": dict(H=4096, N=12288, rot=8192, I=11008, hd=128, sigma=0.02),
    "13b": dict(H=5120, N=15360, rot=10240, I=13824, hd=128, sigma=0.02),
    "30b": dict(H=6656, N=19968, rot=13312, I=17920, hd=128, sigma=0.02),
    "70b": dict(H=8192, N=10240, rot=9216, I=28672, hd=128, sigma=0.015),
}
# query heads, cache heads, head size
HEADS = {"tiny": (8, 8, 64), "7b": (32, 32, 128), "13b": (40, 40, 128), "30b": (52, 52, 128), "70b": (64, 8, 128)}


def _shaped(kind, shape, M, **more):
    return dict(kind=kind, M=M, **SHAPES[shape], **more)


def _attention(shape, B, S, **more):
    Hq, Hkv, D = HEADS[shape]
    return dict(kind="attention", B=B, Hq=Hq, Hkv=Hkv, D=D, S=S, **more)


def listed():
    return [
        # a toy or draft model answering one request: nothing but latency and launches
        _shaped("layer", "tiny", 1, name="layer_tiny_m1"),
        # one interactive request on a small model
        _shaped("layer", "7b", 1, name="layer_7b_m1"),
        # the everyday decode step of a served batch, whole layer with its attention
        _shaped("step", "7b", 32, S=1024, name="step_7b_m32"),
        # half a decode batch through the widest projection in front of attention
        _shaped("qkv", "13b", 16, name="qkv_13b_m16"),
        # a full decode batch through the MLP of a larger model
        _shaped("norm_mlp", "30b", 32, name="norm_mlp_30b_m32"),
        # decode batches beyond 32 requests, or a short chunk of a prompt next to them: odd counts
        _shaped("norm_mlp", "7b", 72, name="norm_mlp_7b_m72"),
        # a short prompt (or several) through QKV
        _shaped("qkv", "7b", 203, name="qkv_7b_m203"),
        # a prompt of ordinary length through the MLP
        _shaped("mlp", "13b", 512, name="mlp_13b_m512"),
        # sizes that fit no tile: a shape of somebody's own, between the regimes
        dict(kind="residual", M=333, N=5001, K=1384, sigma=0.02, name="residual_odd_m333"),
        # a long prompt through a whole layer of the largest model
        _shaped("layer", "70b", 2048, name="layer_70b_m2048"),
        # a served batch, every request at its own length, one cache head per query head
        _attention("7b", 32, 2048, name="attention_7b_b32"),
        # a few long conversations on grouped-query heads
        _attention("70b", 6, 8192, name="attention_70b_b6"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["layer", "step", "qkv", "linear", "residual", "mlp", "norm_mlp", "attention"])
    if kind == "attention":
        case = _attention(rng.choice(list(HEADS)), _log_int(rng, 1, 64), _log_int(rng, 100, 8192))
        while case["B"] * case["Hkv"] * case["S"] * case["D"] > 1 << 28:
            case["S"] = case["S"] // 2
        return case
    if kind == "step":
        return _shaped(kind, rng.choice(["tiny", "7b", "13b", "70b"]), _log_int(rng, 1, 32), S=_log_int(rng, 100, 1024))
    M = _log_int(rng, 1, 2048)
    if kind in ("linear", "residual"):
        if rng.random() < 0.4:      # any sizes: K a multiple of 8, N anything
            return dict(kind=kind, M=M, N=_log_int(rng, 300, 16000), K=8 * _log_int(rng, 32, 1400), sigma=0.02)
        s = SHAPES[rng.choice(list(SHAPES))]
        N, K = rng.choice([(s["H"], s["H"]), (s["H"], s["I"])])
        return dict(kind=kind, M=M, N=N, K=K, sigma=s["sigma"])
    return _shaped(kind, rng.choice(list(SHAPES)), M)


def _lengths(case):
    """Live positions per request: spread evenly from a quarter of the cache to nearly all of it."""
    B, S = case["B"] if case["kind"] == "attention" else case["M"], case["S"]
    lo, hi = max(1, S // 4), max(1, S - S // 50)
    return [hi - (hi - lo) * b // max(1, B - 1) for b in range(B)]


def _inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def normal(*shape, scale=1.0, shift=0.0):
        t = torch.empty(*shape, dtype=torch.float16, device="cuda").normal_(0.0, 1.0, generator=gen)
        if scale != 1.0:
            t.mul_(scale)
        if shift != 0.0:
            t.add_(shift)
        return t

    def lengths():
        order = torch.randperm(len(_lengths(case)), generator=gen, device="cuda")
        return torch.tensor(_lengths(case), dtype=torch.int32, device="cuda")[order].contiguous()

    kind, s = case["kind"], {}
    if kind == "attention":
        B, Hq, Hkv, D, S = case["B"], case["Hq"], case["Hkv"], case["D"], case["S"]
        return dict(q=normal(B, Hq, D), k=normal(B, Hkv, S, D), v=normal(B, Hkv, S, D), lens=lengths())
    M, sigma = case["M"], case["sigma"]
    if kind in ("linear", "residual"):
        s = dict(x=normal(M, case["K"]), w=normal(case["N"], case["K"], scale=sigma))
        if kind == "residual":
            s["res"] = normal(M, case["N"])
        return s
    H, N, I = case["H"], case["N"], case["I"]
    if kind in ("layer", "step", "qkv"):
        s.update(x=normal(M, H), gamma=normal(H, scale=0.1, shift=1.0), w_qkv=normal(N, H, scale=sigma))
    if kind in ("layer", "step"):
        s.update(w_o=normal(H, H, scale=sigma))
    if kind == "layer":
        s.update(a_o=normal(M, H), x_mlp=normal(M, H))
    if kind in ("layer", "step", "mlp", "norm_mlp"):
        s.update(w_gate=normal(I, H, scale=sigma), w_up=normal(I, H, scale=sigma), w_down=normal(H, I, scale=sigma))
    if kind in ("mlp", "norm_mlp"):
        s.update(x=normal(M, H))
    if kind == "norm_mlp":
        s.update(gamma=normal(H, scale=0.1, shift=1.0), res=normal(M, H))
    if kind in ("qkv", "step"):
        s["theta"] = (10000.0 ** (-torch.arange(0, case["hd"], 2, dtype=torch.float64, device="cuda") / case["hd"])).float()
    if kind == "qkv":
        s["pos"] = torch.randint(0, 4096, (M,), dtype=torch.int32, device="cuda", generator=gen)
    if kind == "step":
        Hkv = (N - H) // 2 // case["hd"]
        s.update(gamma2=normal(H, scale=0.1, shift=1.0), lens=lengths(), k=normal(M, Hkv, case["S"], case["hd"]),
                 v=normal(M, Hkv, case["S"], case["hd"]))
        s["pos"] = (s["lens"] - 1).contiguous()          # the new token's position: the last live one
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    kind = case["kind"]

    def out(*shape):
        return torch.empty(*shape, dtype=torch.float16, device="cuda")

    s["case"] = case
    if kind == "attention":
        s["ws"] = thi.Workspace(thi.thi_attention_workspace_bytes(case["B"], case["Hq"], case["Hkv"], case["D"], case["S"]),
                                init=False)
        s["out"] = torch.empty_like(s["q"])
        return s
    M = case["M"]
    if kind in ("linear", "residual"):
        s["ws"] = thi.Workspace.for_ops([(1, M, case["N"], case["K"])])
        s["out"] = out(M, case["N"])
        return s
    H, N, I, hd = case["H"], case["N"], case["I"], case["hd"]
    need = max(thi.thi_workspace_bytes(0, M, N, H), thi.thi_workspace_bytes(1, M, H, H), thi.thi_workspace_bytes(2, M, H, I))
    if kind == "step":
        need = max(need, thi.thi_attention_workspace_bytes(M, H // hd, (N - H) // 2 // hd, hd, case["S"]))
        s.update(rows=torch.arange(M, device="cuda"), at=s["pos"].long(), attn=out(M, H // hd, hd), mid=out(M, H))
    s["ws"] = thi.Workspace(need)
    if kind in ("layer", "step", "qkv"):
        s["qkv"] = out(M, N)
    if kind == "layer":
        s["o"] = out(M, H)
    if kind != "qkv":
        s["out"] = out(M, H)
    return s


def run(s):
    case, ws = s["case"], s["ws"]
    kind = case["kind"]
    if kind == "attention":
        thi.thi_decode_attention(s["q"], s["k"], s["v"], s["lens"], case["D"] ** -0.5, s["out"], ws)
        return [s["out"]]
    if kind == "linear":
        thi.thi_linear(s["x"], s["w"], s["out"], ws)
        return [s["out"]]
    if kind == "residual":
        thi.thi_linear_residual(s["x"], s["w"], s["res"], s["out"], ws)
        return [s["out"]]
    if kind == "mlp":
        thi.thi_swiglu_mlp(s["x"], s["w_gate"], s["w_up"], s["w_down"], s["out"], ws)
        return [s["out"]]
    if kind == "norm_mlp":
        thi.thi_rmsnorm_swiglu_mlp(s["x"], s["gamma"], EPS, s["w_gate"], s["w_up"], s["w_down"], s["res"], s["out"], ws)
        return [s["out"]]
    if kind == "layer":
        thi.thi_rmsnorm_qkv(s["x"], s["gamma"], EPS, s["w_qkv"], s["qkv"], ws)
        thi.thi_linear(s["a_o"], s["w_o"], s["o"], ws)
        thi.thi_swiglu_mlp(s["x_mlp"], s["w_gate"], s["w_up"], s["w_down"], s["out"], ws)
        return [s["qkv"], s["o"], s["out"]]
    thi.thi_rmsnorm_qkv_rope(s["x"], s["gamma"], EPS, s["w_qkv"], s["pos"], s["theta"], case["rot"], case["hd"], s["qkv"], ws)
    if kind == "qkv":
        return [s["qkv"]]
    M, H, N, hd = case["M"], case["H"], case["N"], case["hd"]
    mid = (H + N) // 2
    q = s["qkv"][:, :H].contiguous().view(M, H // hd, hd)
    s["k"][s["rows"], :, s["at"]] = s["qkv"][:, H:mid].view(M, -1, hd)
    s["v"][s["rows"], :, s["at"]] = s["qkv"][:, mid:].view(M, -1, hd)
    thi.thi_decode_attention(q, s["k"], s["v"], s["lens"], hd ** -0.5, s["attn"], ws)
    thi.thi_linear_residual(s["attn"].view(M, H), s["w_o"], s["x"], s["mid"], ws)
    thi.thi_rmsnorm_swiglu_mlp(s["mid"], s["gamma2"], EPS, s["w_gate"], s["w_up"], s["w_down"], s["mid"], s["out"], ws)
    return [s["qkv"], s["attn"], s["mid"], s["out"]]


def work(case):
    kind = case["kind"]
    if kind == "attention":
        live = sum(_lengths(case))
        B, Hq, Hkv, D = case["B"], case["Hq"], case["Hkv"], case["D"]
        return {"bytes": 4 * live * Hkv * D + 4 * B * Hq * D, "flops": 4 * live * Hq * D}
    M = case["M"]

    def linear(n, k):
        return 2 * (n * k + M * k + M * n), 2 * M * n * k

    if kind in ("linear", "residual"):
        b, f = linear(case["N"], case["K"])
        return {"bytes": b + (2 * M * case["N"] if kind == "residual" else 0), "flops": f}
    H, N, I = case["H"], case["N"], case["I"]
    b = f = 0
    if kind in ("layer", "step", "qkv"):
        b, f = linear(N, H)
        b += 2 * H
    if kind in ("layer", "step"):
        ob, of = linear(H, H)
        b, f = b + ob, f + of
    if kind in ("layer", "step", "mlp", "norm_mlp"):
        b, f = b + 2 * (3 * H * I + 2 * M * H), f + 6 * M * H * I
    if kind == "norm_mlp":
        b += 2 * (M * H + H)
    if kind == "step":
        live, Hkv = sum(_lengths(case)), (N - H) // 2 // case["hd"]
        b, f = b + 4 * live * Hkv * case["hd"], f + 4 * live * H
    return {"bytes": b, "flops": f}


def tolerance(case):
    # fp16 storage, fp32 sums: rounding a result once is 2.1e-4 in the mean, x * gamma rounded in front of a projection
    # makes that 2.9e-4, the normalised MLP (x * gamma, h, the result) 4.1e-4, a chain of four operators 4.9e-4.
    # Four times that.
    return {"rel": {"step": 2.0e-3, "norm_mlp": 1.6e-3}.get(case["kind"], 1.2e-3)}


def _norm(x, gamma):
    return x * gamma / torch.sqrt((x * x).mean(dim=1, keepdim=True) + EPS)


def _rope(y, pos, theta, rot, hd):
    ang = pos.double()[:, None] * theta.double()[None, :]
    c, s = torch.cos(ang)[:, None, :], torch.sin(ang)[:, None, :]
    p = y[:, :rot].reshape(y.shape[0], rot // hd, hd // 2, 2)
    a, b = p[..., 0], p[..., 1]
    r = torch.stack((a * c - b * s, b * c + a * s), dim=-1).reshape(y.shape[0], rot)
    return torch.cat((r, y[:, rot:]), dim=1)


def _mlp(x, s):
    h = torch.nn.functional.silu(x @ s["w_gate"].double().t())
    h *= x @ s["w_up"].double().t()
    return h @ s["w_down"].double().t()


def _attend(q, k, v, lens, newest=None):
    """q [B,Hq,D] double; caches fp16; newest: this step's (keys, values) [B,Hkv,D], at the last live position."""
    B, Hq, D = q.shape
    Hkv = k.shape[1]
    out = torch.empty_like(q)
    for b, n in enumerate(lens.tolist()):
        kb, vb = k[b, :, :n].double(), v[b, :, :n].double()
        if newest is not None:
            kb[:, n - 1], vb[:, n - 1] = newest[0][b], newest[1][b]
        for h in range(Hkv):
            qh = q[b, h * (Hq // Hkv):(h + 1) * (Hq // Hkv)]
            p = torch.softmax(qh @ kb[h].t().contiguous() * D ** -0.5, dim=1)
            out[b, h * (Hq // Hkv):(h + 1) * (Hq // Hkv)] = p @ vb[h]
    return out


def exact(case, seed):
    s = _inputs(case, seed)
    kind = case["kind"]
    if kind == "attention":
        return [_attend(s["q"].double(), s["k"], s["v"], s["lens"])]
    x = s["x"].double()
    if kind in ("linear", "residual"):
        y = x @ s["w"].double().t()
        return [y + s["res"].double() if kind == "residual" else y]
    if kind == "mlp":
        return [_mlp(x, s)]
    if kind == "norm_mlp":
        return [_mlp(_norm(x, s["gamma"].double()), s) + s["res"].double()]
    qkv = _norm(x, s["gamma"].double()) @ s["w_qkv"].double().t()
    if kind == "layer":
        return [qkv, s["a_o"].double() @ s["w_o"].double().t(), _mlp(s["x_mlp"].double(), s)]
    qkv = _rope(qkv, s["pos"], s["theta"], case["rot"], case["hd"])
    if kind == "qkv":
        return [qkv]
    M, H, N, hd = case["M"], case["H"], case["N"], case["hd"]
    edge = (H + N) // 2
    k_new, v_new = qkv[:, H:edge].view(M, -1, hd), qkv[:, edge:].view(M, -1, hd)
    attn = _attend(qkv[:, :H].reshape(M, H // hd, hd), s["k"], s["v"], s["lens"], (k_new, v_new))
    mid = x + attn.reshape(M, H) @ s["w_o"].double().t()
    return [qkv, attn, mid, mid + _mlp(_norm(mid, s["gamma2"].double()), s)]
