"""The work that this library does for a program that uses it, as cases that can be timed and checked.

A case is one of two kinds:

* "linear": the forward pass of quantized linear layers, Y = X W^T over K' = K + S.  The activations are quantized
  (with RMSNorm in front where the layer follows one) and multiplied with weights that were packed when the model was
  loaded.  Decode steps (few rows, the weight stream and the launches count) go through the prepared calls and over
  several layers of one shape, each with weights of its own, as a model does; prefills go through the plain calls.
* "offline": what is done once per layer before that: the running channel maxima over calibration batches, the
  channel order and S, and the packing of the weight with them.

S comes out of a threshold on the calibration maxima and is only rounded up to a whole block, so K' is a multiple of the
block (16 for NVFP4, 32 for MXFP4) and mostly no larger power of two.
"""
import math

import numpy as np
import torch

from paper_2601_07475_amd import binding as B

#: A drawn case has at most this many products of a row, a channel and a feature: the largest listed one's.
MOST = 8192 * 8192 * 28672


def _linear(name, fmt, M, K, N, S, norm=False, layers=0, out="f16", interleaved=False, round_up=False):
    return {"name": name, "kind": "linear", "fmt": fmt, "M": M, "K": K, "N": N, "S": S, "norm": norm, "layers": layers,
            "out": out, "interleaved": interleaved, "round_up": round_up}


def listed():
    return [
        # one token of one user: the query projection of an 8B model, the smallest call there is
        _linear("decode_1x4096x4096", "nvfp4", 1, 4096, 4096, 256, layers=1),
        # 16 users decoding: up projection (behind the norm) and down projection of an 8B model, four layers each
        _linear("decode_16x4096x14336_norm", "nvfp4", 16, 4096, 14336, 256, norm=True, layers=4),
        _linear("decode_16x14336x4096", "nvfp4", 16, 14336, 4096, 208, layers=4),
        # a larger batch on a 70B model's up projection
        _linear("decode_32x8192x28672_norm", "nvfp4", 32, 8192, 28672, 272, norm=True, layers=1),
        # a short prompt into the fused q/k/v projection, Appendix D's layout and the scale of the error bound
        _linear("prompt_333x4096x6144_norm", "nvfp4", 333, 4096, 6144, 144, norm=True, interleaved=True, round_up=True),
        # a prompt of 2048 tokens, query projection of an 8B model behind the norm
        _linear("prefill_2048x4096x4096_norm", "nvfp4", 2048, 4096, 4096, 256, norm=True),
        # several prompts together, fused q/k/v projection of a 70B model, rows and K' as they come, fp32 output
        _linear("prefill_1777x8192x10240_f32", "nvfp4", 1777, 8192, 10240, 336, out="f32"),
        # the largest: down projection of a 70B model over 8192 tokens
        _linear("prefill_8192x28672x8192", "nvfp4", 8192, 28672, 8192, 1024),
        # the MXFP4 variant: decode, an MLP of a 32B model, and a prompt with K' as the threshold gives it
        _linear("mx_decode_16x4096x14336", "mx", 16, 4096, 14336, 256, layers=4),
        _linear("mx_prefill_4096x5120x27648", "mx", 4096, 5120, 27648, 512),
        _linear("mx_prefill_1500x4096x14336", "mx", 1500, 4096, 14336, 224),
        # loading a layer: calibration over four batches of 2048 tokens, channel order, S, weight packing
        {"name": "offline_8192x8192", "kind": "offline", "fmt": "nvfp4", "M": 2048, "batches": 4, "K": 8192, "N": 8192},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    fmt = rng.choice(["nvfp4", "nvfp4", "nvfp4", "mx"])
    unit = 16 if fmt == "nvfp4" else 32
    what = rng.choice(["decode", "decode", "prompt", "prefill", "prefill", "offline"])
    K = max(1024, _log(rng, 1024, 28672) // unit * unit)
    N = _log(rng, 1024, 28672)
    if rng.random() < 0.8:
        N = N // 16 * 16
    if what == "offline":
        return {"kind": "offline", "fmt": fmt, "M": _log(rng, 256, 4096), "batches": rng.randint(1, 4), "K": K, "N": N}
    S = min(K, _log(rng, 32, 1024) // unit * unit)
    M = _log(rng, *{"decode": (1, 64), "prompt": (65, 512), "prefill": (513, 8192)}[what])
    while M * K * N > MOST:
        M = M * 3 // 4
    c = _linear("", fmt, M, K, N, S, norm=fmt == "nvfp4" and K <= 16384 and rng.random() < 0.5,
                layers=1 if what == "decode" else 0, out="f32" if rng.random() < 0.2 else "f16",
                interleaved=rng.random() < 0.2, round_up=rng.random() < 0.2)
    del c["name"]
    return c


# ---------------------------------------------------------------------------------------------------------------
# inputs

def _activations(g, rows, K):
    """N(0, 1) with one channel in a hundred 20 to 100 times as large, fp16."""
    f = torch.ones(K, device="cuda")
    heavy = torch.randperm(K, generator=g, device="cuda")[:max(1, K // 100)]
    f[heavy] = torch.exp(math.log(20.0) + math.log(5.0) * torch.rand(heavy.numel(), generator=g, device="cuda"))
    return (torch.randn(rows, K, generator=g, device="cuda") * f).clamp_(-60000.0, 60000.0).half()


def _weights(g, N, K):
    return (0.02 * torch.randn(N, K, generator=g, device="cuda")).half()


def _gamma(g, K):
    """RMSNorm weight: near 1, and a few channels far from it."""
    w = 1.0 + 0.1 * torch.randn(K, generator=g, device="cuda")
    odd = torch.randperm(K, generator=g, device="cuda")[:max(1, K // 128)]
    w[odd] *= torch.tensor([0.05, 0.25, 4.0, 12.0], device="cuda")[torch.randint(4, (odd.numel(),), generator=g, device="cuda")]
    return w.half()


def _scale(t):
    return float(np.float32(float(t.abs().max())) / np.float32(2688.0))


EPS = 1e-5


def _flags(case):
    return (B.LAYOUT_INTERLEAVED if case["interleaved"] else 0) | (B.SCALE_ROUND_UP if case["round_up"] else 0)


def _layer_inputs(case, seed, layer):
    g = torch.Generator(device="cuda").manual_seed(seed * 64 + layer)
    x = _activations(g, case["M"], case["K"])
    w = _weights(g, case["N"], case["K"])
    gamma = _gamma(g, case["K"]) if case["norm"] else None
    # the calibrated order: channels by the largest value seen where the quantizer sees them
    seen = x.float()
    if gamma is not None:
        seen = seen * torch.rsqrt(seen.square().mean(1, keepdim=True) + EPS) * gamma.float()
    perm = torch.sort(seen.abs().amax(0), stable=True).indices.int()
    return x, w, gamma, perm, _scale(seen), _scale(w)


def _pack(case, w, perm, sT_w):
    flags = _flags(case)
    if case["fmt"] == "mx":
        return B.arcq_mx_pack_weight_ex(w, perm, case["S"], flags) if flags else B.arcq_mx_pack_weight(w, perm, case["S"])
    return B.arcq_pack_weight_ex(w, perm, case["S"], sT_w, flags) if flags else B.arcq_pack_weight(w, perm, case["S"], sT_w)


def _dtype(case):
    return torch.float32 if case["out"] == "f32" else torch.float16


def _prepared_layer(case, s):
    """The buffers and prepared calls of one decode layer."""
    M, N, S, Kp = case["M"], case["N"], case["S"], case["K"] + case["S"]
    mx = case["fmt"] == "mx"
    codes = torch.empty((M, Kp // 2), dtype=torch.uint8, device="cuda")
    scales = torch.empty((M, Kp // (32 if mx else 16)), dtype=torch.uint8, device="cuda")
    y = torch.empty((M, N), dtype=_dtype(case), device="cuda")
    need = B.arcq_mx_gemm_workspace_size(M, N, Kp) if mx else B.arcq_gemm_workspace_size(M, N, Kp)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda") if need else None
    flags = _flags(case)
    if mx:
        quantize = (lambda: B.arcq_mx_quantize_act_ex(s["x"], s["perm"], S, flags, codes, scales)) if flags else \
            B.prepare_mx_quantize_act(s["x"], s["perm"], S, codes, scales)
        gemm = B.prepare_mx_gemm(codes, scales, s["wc"], s["ws"], y, ws)
    else:
        if flags and case["norm"]:
            quantize = lambda: B.arcq_rmsnorm_quantize_act_ex(s["x"], s["gamma"], EPS, s["perm"], S, s["sx"], flags, codes, scales)  # noqa: E731
        elif flags:
            quantize = lambda: B.arcq_quantize_act_ex(s["x"], s["perm"], S, s["sx"], flags, codes, scales)  # noqa: E731
        elif case["norm"]:
            quantize = B.prepare_rmsnorm_quantize_act(s["x"], s["gamma"], EPS, s["perm"], S, s["sx"], codes, scales)
        else:
            quantize = B.prepare_quantize_act(s["x"], s["perm"], S, s["sx"], codes, scales)
        gemm = B.prepare_gemm(codes, scales, s["sx"], s["wc"], s["ws"], s["sw"], y, ws)
    return {"quantize": quantize, "gemm": gemm, "out": {"codes": codes, "scales": scales, "y": y}, "keep": (s, ws)}


def prepare(case, seed):
    if case["kind"] == "offline":
        g = torch.Generator(device="cuda").manual_seed(seed * 64)
        f = torch.ones(case["K"], device="cuda")
        f[torch.randperm(case["K"], generator=g, device="cuda")[:max(1, case["K"] // 100)]] = 50.0
        x = [(torch.randn(case["M"], case["K"], generator=g, device="cuda") * f).clamp_(-60000.0, 60000.0).half()
             for _ in range(case["batches"])]
        w = _weights(g, case["N"], case["K"])
        return {"case": case, "x": x, "w": w, "sw": _scale(w)}
    layers = []
    for layer in range(max(1, case["layers"])):
        x, w, gamma, perm, sx, sw = _layer_inputs(case, seed, layer)
        wc, ws = _pack(case, w, perm, sw)
        layers.append({"x": x, "gamma": gamma, "perm": perm, "sx": sx, "sw": sw, "wc": wc, "ws": ws})
    if case["layers"]:
        return {"case": case, "layers": [_prepared_layer(case, s) for s in layers]}
    if case["fmt"] == "mx":     # the workspace that a program keeps for this shape
        need = B.arcq_mx_gemm_workspace_size(case["M"], case["N"], case["K"] + case["S"])
        layers[0]["workspace"] = torch.empty(need, dtype=torch.uint8, device="cuda") if need else None
    return {"case": case, **layers[0]}


# ---------------------------------------------------------------------------------------------------------------
# one pass

def _run_offline(s):
    case = s["case"]
    colmax = torch.zeros(case["K"], dtype=torch.float32, device="cuda")
    for xb in s["x"]:
        B.arcq_calib_absmax(xb, colmax)
    perm, S, info = B.arcq_calib_select(colmax)
    if case["fmt"] == "mx":
        S = min(case["K"], -(-S // 32) * 32)
        codes, scales = B.arcq_mx_pack_weight(s["w"], perm, S)
    else:
        codes, scales = B.arcq_pack_weight(s["w"], perm, S, s["sw"])
    return {"colmax": colmax, "perm": perm, "S": S, "info": info, "codes": codes, "scales": scales}


def run(s):
    case = s["case"]
    if case["kind"] == "offline":
        return _run_offline(s)
    if case["layers"]:
        for layer in s["layers"]:
            layer["quantize"]()
            layer["gemm"]()
        return [layer["out"] for layer in s["layers"]]
    S, flags = case["S"], _flags(case)
    if case["fmt"] == "mx":
        if flags:
            codes, scales = B.arcq_mx_quantize_act_ex(s["x"], s["perm"], S, flags)
        else:
            codes, scales = B.arcq_mx_quantize_act(s["x"], s["perm"], S)
        y = B.arcq_mx_gemm(codes, scales, s["wc"], s["ws"], out_dtype=_dtype(case), workspace=s["workspace"])
    else:
        if case["norm"] and flags:
            codes, scales = B.arcq_rmsnorm_quantize_act_ex(s["x"], s["gamma"], EPS, s["perm"], S, s["sx"], flags)
        elif case["norm"]:
            codes, scales = B.arcq_rmsnorm_quantize_act(s["x"], s["gamma"], EPS, s["perm"], S, s["sx"])
        elif flags:
            codes, scales = B.arcq_quantize_act_ex(s["x"], s["perm"], S, s["sx"], flags)
        else:
            codes, scales = B.arcq_quantize_act(s["x"], s["perm"], S, s["sx"])
        y = B.arcq_gemm(codes, scales, s["sx"], s["wc"], s["ws"], s["sw"], out_dtype=_dtype(case))
    return {"codes": codes, "scales": scales, "y": y}


# ---------------------------------------------------------------------------------------------------------------
# what a pass cannot do without, and how far two correct results may be apart

def work(case):
    K, N, M = case["K"], case["N"], case["M"]
    if case["kind"] == "offline":
        # batches and weight read, maxima, order and packed weight written (S is about a hundredth of K)
        per = 9 / 16 if case["fmt"] == "nvfp4" else 17 / 32
        return {"bytes": 2 * K * (M * case["batches"] + N) + 12 * K + N * K * per, "flops": 0}
    Kp = K + case["S"]
    per = 9 / 16 if case["fmt"] == "nvfp4" else 17 / 32
    one = 2 * M * K + 4 * K + (2 * K if case["norm"] else 0) + M * Kp * per + N * Kp * per + M * N * (4 if case["out"] == "f32" else 2)
    return {"bytes": one * max(1, case["layers"]), "flops": 2 * M * N * Kp * max(1, case["layers"])}


def tolerance(case):
    """Codes and scale bytes are the same bit for bit.  The product is summed in fp32 in any order and rounded once to
    fp16 or kept in fp32.  Measured against 64 bits, 2-norms: NVFP4 1e-7 in fp32 and 2.1e-4 after the rounding to fp16; the
    scaled FP4 matrix instruction of MXFP4 keeps fewer bits inside one instruction, 1.5e-4 before the rounding, 2.6e-4 after."""
    if case["kind"] == "offline":
        return "exact"
    if case["fmt"] == "mx":
        return {"rel": 1e-3, "max": 6e-3}
    return {"rel": 1e-6, "max": 4e-5} if case["out"] == "f32" else {"rel": 8e-4, "max": 4e-3}


# ---------------------------------------------------------------------------------------------------------------
# the same in 64 bits: the fp32 steps that decide on a code are rounded to fp32 one by one, as the format says

def _r32(t):
    return t.float().double()


def _pow2(e):
    return torch.ldexp(torch.ones((), dtype=torch.float64, device="cuda"), e)


def _e2m1(w):
    """The nearest value of the E2M1 grid, ties to the even mantissa, saturating at 6."""
    a = w.abs()
    step = torch.where(a < 2, 0.5, torch.where(a < 4, 1.0, 2.0))
    return torch.sign(w) * (torch.round(a / step) * step).clamp_(max=6.0)


def _stage_nvfp4(v, sT, up):
    """One quantization of blocks v [..., 16]: (values without the tensor scale, residual)."""
    ginv = float(np.float32(1.0) / np.float32(np.float32(6.0) * np.float32(sT)))
    u = _r32(v.abs().amax(-1, keepdim=True) * ginv)
    step = _pow2(torch.clamp(torch.frexp(u).exponent - 1, min=-6) - 3)
    e4m3 = ((torch.ceil if up else torch.round)(u / step) * step).clamp(max=448.0)
    s = _r32(e4m3 * float(np.float32(sT)))
    inv = torch.where(s > 0, _r32(1.0 / s.clamp(min=1e-300)), torch.zeros_like(s))
    q = _e2m1(_r32(v * inv))
    return q * e4m3, _r32(v - s * q)


def _stage_mx(v, up):
    amax = v.abs().amax(-1, keepdim=True)
    X = _pow2(torch.frexp(amax).exponent - 3)
    if up:
        X = torch.where(amax > 6 * X, 2 * X, X)
    X = torch.where(amax > 0, X, torch.ones_like(X))
    q = _e2m1(v / X)
    return q * X, v - q * X


def _operand(case, t, perm, sT, weight, norm=None):
    """The dequantized operand [rows, K'] in 64 bits, without its tensor scale."""
    rows, K = t.shape
    S, bs = case["S"], 32 if case["fmt"] == "mx" else 16
    out = torch.empty((rows, K + S), dtype=torch.float64, device="cuda")
    for r0 in range(0, rows, 1024):
        v = t[r0:r0 + 1024].double()
        n = v.shape[0]
        if norm is not None:
            ms = _r32(v.square().mean(1, keepdim=True))
            rstd = _r32(1.0 / _r32(torch.sqrt(_r32(ms + float(np.float32(EPS))))))
            v = (_r32(v * rstd).half().double() * norm.double()).half().double()
        v = v[:, perm.long()].view(n, K // bs, bs)
        q, res = _stage_nvfp4(v, sT, case["round_up"]) if bs == 16 else _stage_mx(v, case["round_up"])
        o0 = (K - S) // bs
        if weight:
            tail = q[:, o0:]
        else:
            tail = (_stage_nvfp4(res[:, o0:], sT, case["round_up"]) if bs == 16 else _stage_mx(res[:, o0:], case["round_up"]))[0]
        out[r0:r0 + 1024, :K] = q.reshape(n, K)
        out[r0:r0 + 1024, K:] = tail.reshape(n, S)
    return out


def exact(case, seed):
    if case["kind"] == "offline":
        s = prepare(case, seed)
        colmax = torch.stack([xb.abs().amax(0) for xb in s["x"]]).amax(0).double()
        return {"colmax": colmax, "perm": None, "S": None, "info": None, "codes": None, "scales": None}
    got = []
    for layer in range(max(1, case["layers"])):
        x, w, gamma, perm, sx, sw = _layer_inputs(case, seed, layer)
        a = _operand(case, x, perm, sx, False, gamma)
        b = _operand(case, w, perm, sw, True)
        alpha = 1.0 if case["fmt"] == "mx" else float(np.float32(sx)) * float(np.float32(sw))
        got.append({"codes": None, "scales": None, "y": (a @ b.t()) * alpha})
    return got if case["layers"] else got[0]
