"""Performance cases of the K-interval attention library.

Each case is one call pattern of a user's program, through the public entry
points of ``paper_2609_33591_amd``:

``step``      one training step with buffers the program keeps (o, stats, dq,
              dk, dv): ``kia_attn_fwd*`` then ``kia_attn_bwd*``;
``autograd``  the operation inside a model: ``k_interval_attention`` and
              ``torch.autograd.grad``;
``eval``      ``k_interval_attention`` under ``torch.no_grad``.

``dtype`` is the input and output type: ``f32``, ``bf16`` (bfloat16 inputs,
float32 outputs) or ``bf16o`` (bfloat16 in and out). Inputs are N(0,1) draws
(q and k times ``qk``), the inputs of this repository's benchmark.
"""
import math

import torch

import paper_2609_33591_amd as kia

_OP = dict(K=4, calib="fwm", tau=8.0, recon="nearest", ste="prob", detach="full", causal=True,
           qk=1.0)


def _case(name, kind, dtype, B, H, T, d, **op):
    return dict(_OP, name=name, kind=kind, dtype=dtype, B=B, H=H, T=T, d=d, **op)


def listed():
    return [
        # the smallest call: one head of 64 keys (smoke runs, unit tests)
        _case("tiny_step", "step", "f32", 1, 1, 64, 16, calib="minmax", recon="lerp", ste="weight"),
        # the paper's own training call: micro-batch 1 of the 124M model, inside the model
        _case("mb1_124m_autograd", "autograd", "f32", 1, 12, 1024, 64),
        # the same of the 1B model, in bf16 autocast
        _case("mb1_1b_bf16o_autograd", "autograd", "bf16o", 1, 24, 1024, 64),
        # a ragged batch of a small model: T no multiple of a tile, an odd K
        _case("ragged_d32_step", "step", "f32", 3, 5, 777, 32, K=7, calib="minmax", ste="weight"),
        # GPT-2-124M attention, batch 8: the benchmark step
        _case("gpt2_124m_step", "step", "f32", 8, 12, 1024, 64),
        # the same shape with the paper's MinMax LERP baseline
        _case("gpt2_124m_minmax_lerp", "step", "f32", 8, 12, 1024, 64, calib="minmax",
              recon="lerp", ste="weight"),
        # the exact-softmax baseline through the same kernels
        _case("gpt2_124m_softmax", "step", "f32", 8, 12, 1024, 64, recon="softmax"),
        # evaluation forward of the 124M model
        _case("gpt2_124m_eval", "eval", "f32", 8, 12, 1024, 64),
        # every key valid (an encoder), bf16 inputs, ragged length
        _case("encoder_bf16_step", "step", "bf16", 4, 12, 1500, 64, K=16, recon="lerp",
              causal=False),
        # the 1B-scale workload, bf16 inputs
        _case("scale_1b_bf16_step", "step", "bf16", 4, 16, 2048, 128, K=16),
        # its evaluation forward, bf16 in and out
        _case("scale_1b_bf16o_eval", "eval", "bf16o", 4, 16, 2048, 128, K=16),
        # long context, fp32, MinMax LERP, scores twice as wide
        _case("long_8k_step", "step", "f32", 1, 16, 8192, 128, calib="minmax", recon="lerp",
              ste="weight", qk=2.0),
    ]


_MOST = 16 * 8192 * 8192 * 128  # B H T^2 d of the largest listed case


def draw(rng):
    """One more case: sizes spread over the logarithm of their range."""
    kind = rng.choice(("step", "step", "autograd", "eval"))
    dtype = rng.choice(("f32", "f32", "bf16", "bf16o")) if kind == "step" else \
        rng.choice(("f32", "bf16o"))
    d = rng.choice((16, 32, 64, 64, 128))
    causal = rng.random() < 0.8
    T = int(round(math.exp(rng.uniform(math.log(64), math.log(8192)))))
    if rng.random() < 0.4:  # the lengths models are trained at
        T = max(64, (T + 63) // 64 * 64)
    bh = int(round(math.exp(rng.uniform(0.0, math.log(128)))))
    bh = max(1, min(bh, (_MOST if causal else _MOST // 2) // (4 * T * T * d)))
    B = rng.choice([b for b in range(1, bh + 1) if bh % b == 0])
    recon = rng.choice(("lerp", "nearest", "nearest", "softmax") if dtype == "f32"
                       else ("lerp", "nearest", "nearest"))
    return dict(kind=kind, dtype=dtype, B=B, H=bh // B, T=T, d=d,
                K=rng.choice((2, 4, 4, 7, 16, 32)), calib=rng.choice(("minmax", "fwm", "fwm")),
                tau=rng.choice((6.0, 8.0)), recon=recon, ste=rng.choice(("weight", "prob")),
                detach=rng.choice(("full", "full", "detach")), causal=causal,
                qk=rng.choice((0.7, 1.0, 1.5, 2.0)))


def _inputs(case, seed):
    """q, k, v, dO on the GPU, in the case's input type."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 7919 + 17)
    shape = (case["B"], case["H"], case["T"], case["d"])
    x = [torch.randn(shape, generator=g, device="cuda", dtype=torch.float32) for _ in range(4)]
    x[0] *= case["qk"]
    x[1] *= case["qk"]
    return x if case["dtype"] == "f32" else [t.to(torch.bfloat16) for t in x]


def _op(case):
    return (case["K"], case["calib"], case["tau"], case["recon"], case["ste"], case["detach"],
            case["causal"])


def prepare(case, seed):
    q, k, v, dO = _inputs(case, seed)
    s = dict(kind=case["kind"], op=_op(case), q=q, k=k, v=v)
    if case["kind"] == "step":
        b16o = case["dtype"] == "bf16o"
        out = torch.bfloat16 if b16o else torch.float32
        s["stats"] = kia.new_stats(*q.shape, case["recon"], case["ste"], case["causal"],
                                   device=q.device, bf16_out=b16o)
        for n in ("o", "dq", "dk", "dv"):
            s[n] = torch.empty(q.shape, dtype=out, device=q.device)
        s["dO"] = dO
        s["fwd"], s["bwd"] = {
            "f32": (kia.kia_attn_fwd, kia.kia_attn_bwd),
            "bf16": (kia.kia_attn_fwd_bf16, kia.kia_attn_bwd_bf16),
            "bf16o": (kia.kia_attn_fwd_bf16o, kia.kia_attn_bwd_bf16o)}[case["dtype"]]
    elif case["kind"] == "autograd":
        for n in ("q", "k", "v"):
            s[n] = s[n].requires_grad_()
        s["dO"] = dO
    return s


def run(s):
    K, calib, tau, recon, ste, detach, causal = s["op"]
    if s["kind"] == "step":
        s["fwd"](s["q"], s["k"], s["v"], s["o"], s["stats"], *s["op"])
        s["bwd"](s["q"], s["k"], s["v"], s["o"], s["dO"], s["stats"], s["dq"], s["dk"], s["dv"],
                 *s["op"])
        return {n: s[n] for n in ("o", "dq", "dk", "dv")}
    if s["kind"] == "autograd":
        o = kia.k_interval_attention(s["q"], s["k"], s["v"], *s["op"])
        dq, dk, dv = torch.autograd.grad(o, (s["q"], s["k"], s["v"]), s["dO"])
        return {"o": o.detach(), "dq": dq, "dk": dk, "dv": dv}
    with torch.no_grad():
        o = kia.k_interval_attention(s["q"], s["k"], s["v"], K, calib, tau, recon, ste,
                                     causal=causal)
    return {"o": o}


def work(case):
    """Two products forward (Q K^T, P V) and five backward (S or its stored
    form, dP, dV, dQ, dK) over the valid (query, key) pairs; inputs read and
    outputs written once."""
    n = case["B"] * case["H"] * case["T"] * case["d"]
    pairs = case["T"] * (case["T"] + 1) // 2 if case["causal"] else case["T"] ** 2
    unit = 2 * case["B"] * case["H"] * pairs * case["d"]
    i = 4 if case["dtype"] == "f32" else 2
    o = 2 if case["dtype"] == "bf16o" else 4
    if case["kind"] == "eval":
        return {"bytes": n * (3 * i + o), "flops": 2 * unit}
    return {"bytes": n * (4 * i + 4 * o), "flops": 7 * unit}


def tolerance(case):
    """Nearest jumps at a level's midpoint and every gradient at a grid
    point, so a pair whose score lies within rounding of one may differ as a
    whole: against 64 bits 2e-4 to 1.2e-3 in float32 (most at T = 8192 with
    the wide scores). bfloat16 products and outputs show 2e-3 to 3e-3, the
    exact softmax (no jumps) up to 7e-7. About four times that."""
    if case["dtype"] != "f32":
        return {"rel": 1e-2, "max": 0.9}
    if case["recon"] == "softmax":
        return {"rel": 3e-6, "max": 3e-4}
    return {"rel": 5e-3, "max": 0.9}


# ---- the same in 64 bits -------------------------------------------------
def _slice(c, q, k, v, dO, scale):
    """One (b, h) slice: fp64 products, the operator's fp32 scores (the dot
    product and its scaling each rounded once), fp64 from there on."""
    T, K, tau = c["T"], c["K"], c["tau"]
    s32 = (q @ k.T).float() * torch.tensor(scale, dtype=torch.float32, device=q.device)
    valid = torch.ones(T, T, dtype=torch.bool, device=q.device)
    if c["causal"]:
        valid = valid.tril()
    s = s32.double()
    M = s.masked_fill(~valid, -math.inf).amax(1, keepdim=True)
    minmax = c["calib"] == "minmax" and c["recon"] != "softmax"
    m = s.masked_fill(~valid, math.inf).amin(1, keepdim=True) if minmax else M
    on = valid
    if c["recon"] == "softmax":
        w = torch.exp((s32 - M.float()).double())
        w = torch.where(on, w, torch.zeros_like(w))
        wL = wX = Delta = w
    else:
        if minmax:
            degen = (M - m) <= 1e-12
            span = torch.where(degen, torch.ones_like(M), M - m)
            u = K * (s - m) / span
            h, z0 = span / K, -span
        else:
            a = (s - M) + tau
            on = on & (a >= 0)
            u, h, z0 = K * a / tau, tau / K, -tau
        r = u.floor().clamp(0, K - 1)
        t = (u - r).clamp(0, 1)
        del s
        E0, E1 = torch.exp(z0 + r * h), torch.exp(z0 + (r + 1) * h)
        Delta = (E1 - E0) / h
        wL = E0 + t * (E1 - E0)
        w = torch.where(t >= 0.5, E1, E0) if c["recon"] == "nearest" else wL
        if minmax:
            wL, w, Delta = (torch.where(degen, torch.full_like(x, f), x)
                            for x, f in ((wL, 1.0), (w, 1.0), (Delta, 0.0)))
        z = torch.zeros((), dtype=torch.float64, device=q.device)
        wL, w, Delta = (torch.where(on, x, z) for x in (wL, w, Delta))
        wX = w if (c["recon"] == "nearest" and c["ste"] == "weight") else wL
    W = w.sum(1, keepdim=True)
    o = (w / W) @ v
    if dO is None:
        return o, None, None, None
    g = dO @ v.T
    WX = wX.sum(1, keepdim=True)
    gamma = (g - (wX * g).sum(1, keepdim=True) / WX) / WX
    del g
    dv = (w / W).T @ dO
    dS = gamma * Delta
    if c["detach"] == "full":
        ss = dS.sum(1, keepdim=True)
        atM = valid & (s32.double() == M)
        if minmax:
            X = (r * wL + t * E1) / K
            cM = torch.where(on & ~degen, gamma * (X - wL - Delta * (r + t) / K),
                             torch.zeros_like(wL)).sum(1, keepdim=True)
            atm = valid & (s32.double() == m)
            cm = torch.where(degen, torch.zeros_like(ss), -(ss + cM))
            dS = dS + torch.where(atm, cm / atm.sum(1, keepdim=True), torch.zeros_like(dS))
        else:
            cM = -ss
        dS = dS + torch.where(atM, cM / atM.sum(1, keepdim=True), torch.zeros_like(dS))
    return o, scale * (dS @ k), scale * (dS.T @ q), dv


def exact(case, seed):
    if case["B"] * case["H"] * case["T"] ** 2 > 3e9:
        return None
    q, k, v, dO = (x.double() for x in _inputs(case, seed))
    scale = torch.tensor(1.0 / math.sqrt(case["d"]), dtype=torch.float32).item()
    back = case["kind"] != "eval"
    names = ("o", "dq", "dk", "dv") if back else ("o",)
    out = {n: torch.empty_like(q) for n in names}
    for b in range(case["B"]):
        for h in range(case["H"]):
            r = _slice(case, q[b, h], k[b, h], v[b, h], dO[b, h] if back else None, scale)
            for n, x in zip(names, r):
                out[n][b, h] = x
    return out
