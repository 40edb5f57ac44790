"""The work that a program hands to this library, as measurable cases.

Sizes are the library's own workload configurations (Llama-3-8B and 32B-class linear layers, whole
or as the tensor-parallel shards of them that one GPU of a group holds) at the token counts where
such a program runs them: prefill chunks from a few dozen tokens to a long context, decode batches
from one request upwards, and the preparation of the weights at load time.  Four kinds of case:

  linear   the prefill linear layer(s): quantize the activations, block-scaled product (nvfp4_linear),
           with a calibrated tensor-level scale or (dynamic) one computed in the pass
  mlp      the MLP half of a decoder block as a dependent chain with the fused quantizers
  bf16     the product in the precision that decoding keeps (bf16_gemm_ws)
  weights  a weight matrix brought into the form that the product streams

Inputs are drawn on the GPU from the seed, by the recipe of workloads.py (normal activations with
0.1 % outlier channels, Student-t input of the down projection, normal weights of std K^-1/2).
"""
import math

import torch

import paper_2605_20315_amd as mq

# (K, N) of the four linear layers of a block; a tensor-parallel shard splits N of qkv and gate_up,
# K of o and down
MODELS = {
    "llama8b": {"qkv": (4096, 6144), "o": (4096, 4096), "gate_up": (4096, 28672), "down": (14336, 4096)},
    "dense32b": {"qkv": (5120, 7168), "o": (5120, 5120), "gate_up": (5120, 51200), "down": (25600, 5120)},
}
OUTLIER_GAIN = {"llama8b": 20.0, "dense32b": 50.0}
BLOCK = "qkv,o,gate_up,down"
RMS_EPS = 1e-6
# calibrated tensor-level scales of the two activations inside the MLP chain (largest value / 2688)
MLP_ALPHA_IN, MLP_ALPHA_MID = 100.0 / 2688.0, 30.0 / 2688.0
# a program keeps one workspace per stream: the largest that the library asks for
NVFP4_WORKSPACE, BF16_WORKSPACE = 4 << 20, 16 << 20


def _linear(M, layers, model="llama8b", tp=1, dynamic=False, layout="ktile", out="bf16"):
    return {"kind": "linear", "M": M, "model": model, "layers": layers, "tp": tp, "dynamic": dynamic,
            "layout": layout, "out": out}


def _mlp(M, model="llama8b", tp=1):
    return {"kind": "mlp", "M": M, "model": model, "tp": tp}


def _bf16(M, layers, model="llama8b", tp=1, out="bf16"):
    return {"kind": "bf16", "M": M, "model": model, "layers": layers, "tp": tp, "out": out}


def _weights(layer, model="llama8b", tp=1):
    return {"kind": "weights", "layer": layer, "model": model, "tp": tp}


def listed():
    return [
        # one short prompt through one square layer: the smallest call, all latency
        dict(_linear(64, "o"), name="chunk64_o"),
        # a short prefill chunk through the linear layers of a block
        dict(_linear(128, BLOCK), name="chunk128_block"),
        # a chunk of an odd length, as chunked prefill leaves behind
        dict(_linear(333, BLOCK), name="chunk333_block"),
        # the MLP half of a block at an ordinary prompt length, quantizers fused with their producers
        dict(_mlp(1000), name="mlp1000"),
        # one 2048-token chunk through the attention input projection of the larger model
        dict(_linear(2048, "qkv", model="dense32b"), name="prefill2048_32b_qkv"),
        # the last chunk of a ragged multi-turn batch, long K, tensor-level scale computed on the fly
        dict(_linear(5003, "down", dynamic=True), name="ragged5003_down_dynamic"),
        # the widest layer at the long-context chunk size: the largest call
        dict(_linear(8192, "gate_up"), name="prefill8192_gate_up"),
        # decoding one request, a middling batch, a large continuous batch
        dict(_bf16(1, BLOCK), name="decode1_block"),
        dict(_bf16(48, BLOCK), name="decode48_block"),
        dict(_bf16(200, BLOCK), name="decode200_block"),
        # prefill kept in BF16: what the quantized path is compared with
        dict(_bf16(4096, "qkv"), name="bf16_prefill4096_qkv"),
        # loading a weight matrix: scale, canonical NVFP4 bytes, the order that the product streams
        dict(_weights("gate_up"), name="load_gate_up"),
    ]


def _shape(case, layer):
    K, N = MODELS[case["model"]][layer]
    return (K // case["tp"], N) if layer in ("o", "down") else (K, N // case["tp"])


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


LARGEST_FLOPS = 2.0 * 8192 * 4096 * 28672


def draw(rng):
    """One more case of the same ranges: token counts spread over their logarithm, whole layers and
    shards of both models, the options that are in use."""
    while True:
        kind = rng.choice(["linear", "linear", "linear", "linear", "mlp", "bf16", "bf16", "bf16", "weights"])
        model, tp = rng.choice(["llama8b", "llama8b", "dense32b"]), rng.choice([1, 1, 2, 4, 8])
        layers = rng.choice(["qkv", "o", "gate_up", "down", BLOCK])
        if kind == "linear":
            case = _linear(_log_int(rng, 16, 16384), layers, model, tp, dynamic=rng.random() < 0.25,
                           layout="linear" if rng.random() < 0.25 else "ktile",
                           out="fp32" if rng.random() < 0.15 else "bf16")
        elif kind == "mlp":
            case = _mlp(_log_int(rng, 16, 4096), model, tp)
        elif kind == "bf16":
            case = _bf16(_log_int(rng, 1, 4096), layers, model, tp, out="fp32" if rng.random() < 0.15 else "bf16")
        else:
            case = _weights(rng.choice(["qkv", "o", "gate_up", "down"]), model, tp)
        if work(case)["flops"] <= LARGEST_FLOPS and work(case)["bytes"] <= 2.0e9:
            return case


# ---- inputs ---------------------------------------------------------------------------------------

def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _activation(g, M, K, gain, heavy):
    x = torch.randn((M, K), device="cuda", generator=g)
    if heavy:  # Student-t with four degrees of freedom
        chi = torch.zeros_like(x)
        for _ in range(4):
            chi += torch.randn((M, K), device="cuda", generator=g) ** 2
        x /= torch.sqrt(chi / 4.0)
    cols = torch.randperm(K, device="cuda", generator=g)[:max(1, round(K * 1e-3))]
    x[:, cols] *= gain
    return x.to(torch.bfloat16)


def _weight(g, N, K):
    return (torch.randn((N, K), device="cuda", generator=g) * K ** -0.5).to(torch.bfloat16)


def _tensors(case, seed):
    """The BF16 tensors of a case, as both prepare() and exact() start from."""
    g, gain = _generator(seed), OUTLIER_GAIN[case["model"]]
    if case["kind"] == "weights":
        K, N = _shape(case, case["layer"])
        return {"w": _weight(g, N, K)}
    if case["kind"] == "mlp":
        (K1, N1), (K2, N2) = _shape(case, "gate_up"), _shape(case, "down")
        return {"x": _activation(g, case["M"], K1, gain, False),
                "norm": (1.0 + 0.1 * torch.randn(K1, device="cuda", generator=g)).to(torch.bfloat16),
                "w1": _weight(g, N1, K1), "w2": _weight(g, N2, K2)}
    pairs = []
    for layer in case["layers"].split(","):
        K, N = _shape(case, layer)
        heavy = layer == "down" and case["model"] == "llama8b"
        pairs.append((_activation(g, case["M"], K, gain, heavy), _weight(g, N, K)))
    return {"pairs": pairs}


def _nvfp4_weight(w, layout):
    alpha = mq.nvfp4_global_scale(w)
    return mq.nvfp4_quantize(w, alpha, layout=layout) + (alpha,)


def _out(case):
    return (mq.MQ_OUT_FP32, torch.float32) if case["out"] == "fp32" else (mq.MQ_OUT_BF16, torch.bfloat16)


def _empty(shape, dtype):
    return torch.empty(shape, dtype=dtype, device="cuda")


def prepare(case, seed):
    mq.mq_init()
    t = _tensors(case, seed)
    kind = case["kind"]
    if kind == "weights":
        return {"kind": kind, "w": t["w"]}
    M = case["M"]
    u8 = torch.uint8
    if kind == "bf16":
        flag, dtype = _out(case)
        return {"kind": kind, "out": flag, "ws": _empty(BF16_WORKSPACE, u8),
                "layers": [(x, w, _empty((M, w.shape[0]), dtype)) for x, w in t["pairs"]]}
    if kind == "linear":
        flag, dtype = _out(case)
        layout = mq.MQ_LAYOUT_LINEAR if case["layout"] == "linear" else mq.MQ_LAYOUT_KTILE
        layers = []
        for x, w in t["pairs"]:
            N, K = w.shape
            layers.append((x, mq.nvfp4_global_scale(x), _nvfp4_weight(w, layout), _empty((M, N), dtype),
                           _empty((M, K // 2), u8), _empty((M, K // 16), u8)))
        return {"kind": kind, "out": flag, "layout": layout, "dynamic": case["dynamic"],
                "ws": _empty(NVFP4_WORKSPACE, u8), "layers": layers}
    (N1, K1), (N2, K2) = t["w1"].shape, t["w2"].shape
    return {"kind": kind, "x": t["x"], "norm": t["norm"], "ws": _empty(NVFP4_WORKSPACE, u8),
            "a1": torch.full((1,), MLP_ALPHA_IN, device="cuda"), "a2": torch.full((1,), MLP_ALPHA_MID, device="cuda"),
            "w1": _nvfp4_weight(t["w1"], mq.MQ_LAYOUT_KTILE), "w2": _nvfp4_weight(t["w2"], mq.MQ_LAYOUT_KTILE),
            "c1": _empty((M, K1 // 2), u8), "s1": _empty((M, K1 // 16), u8),
            "c2": _empty((M, K2 // 2), u8), "s2": _empty((M, K2 // 16), u8),
            "y1": _empty((M, N1), torch.bfloat16), "y2": _empty((M, N2), torch.bfloat16)}


# ---- one pass -------------------------------------------------------------------------------------

def run(s):
    kind = s["kind"]
    if kind == "linear":
        ys = []
        for x, alpha, (wc, ws, wa), y, codes, scales in s["layers"]:
            if s["dynamic"]:
                mq.nvfp4_global_scale(x, alpha)
            ys.append(mq.nvfp4_linear(x, alpha, wc, ws, wa, s["out"], y, codes, scales, s["layout"], s["ws"]))
        return ys
    if kind == "bf16":
        return [mq.bf16_gemm_ws(x, w, s["ws"], s["out"], y) for x, w, y in s["layers"]]
    kt = mq.MQ_LAYOUT_KTILE
    if kind == "weights":
        alpha = mq.nvfp4_global_scale(s["w"])
        codes, scales = mq.nvfp4_quantize(s["w"], alpha)
        kcodes, kscales = mq.nvfp4_relayout(codes, scales, mq.MQ_LAYOUT_LINEAR, kt)
        return {"alpha": alpha, "codes": codes, "scales": scales, "kcodes": kcodes, "kscales": kscales}
    (w1c, w1s, w1a), (w2c, w2s, w2a) = s["w1"], s["w2"]
    mq.nvfp4_quantize_rmsnorm(s["x"], s["norm"], RMS_EPS, s["a1"], s["c1"], s["s1"], kt)
    mq.nvfp4_gemm_ws(s["c1"], s["s1"], s["a1"], w1c, w1s, w1a, s["ws"], mq.MQ_OUT_BF16, s["y1"], kt)
    mq.nvfp4_quantize_silu_mul(s["y1"], s["a2"], s["c2"], s["s2"], kt)
    mq.nvfp4_gemm_ws(s["c2"], s["s2"], s["a2"], w2c, w2s, w2a, s["ws"], mq.MQ_OUT_BF16, s["y2"], kt)
    return {"gate_up": s["y1"], "down": s["y2"]}


# ---- what a pass cannot do without ----------------------------------------------------------------

def work(case):
    nvfp4 = 0.5 + 1.0 / 16.0  # bytes per element
    if case["kind"] == "weights":
        K, N = _shape(case, case["layer"])
        return {"bytes": N * K * (2.0 + 2.0 * nvfp4), "flops": 0.0}
    M = case["M"]
    if case["kind"] == "mlp":
        (K1, N1), (K2, N2) = _shape(case, "gate_up"), _shape(case, "down")
        return {"bytes": 2.0 * M * K1 + 2.0 * K1 + nvfp4 * (N1 * K1 + N2 * K2) + 2.0 * M * (N1 + N2),
                "flops": 2.0 * M * (N1 * K1 + N2 * K2)}
    size = 4.0 if case["out"] == "fp32" else 2.0
    got = {"bytes": 0.0, "flops": 0.0}
    for layer in case["layers"].split(","):
        K, N = _shape(case, layer)
        got["bytes"] += 2.0 * M * K + N * K * (2.0 if case["kind"] == "bf16" else nvfp4) + size * M * N
        got["flops"] += 2.0 * M * N * K
    return got


def tolerance(case):
    kind = case["kind"]
    if kind == "weights":  # bytes and one IEEE quotient: nothing to differ in
        return "exact"
    # four times what the comparison with exact() shows: 1.7e-3 for the rounding to BF16 (half an ulp at
    # most, 4e-3 of a value), up to 4e-7 for sums kept in binary32; in the chain a gate_up output
    # that rounds the other way can also turn a code of the down projection's input
    if kind == "mlp":
        return {"rel": 1e-2}
    if case["out"] == "fp32":
        return {"rel": 2e-6}
    return {"rel": 7e-3, "max": 1.6e-2}


# ---- the same in 64 bits, plain torch -------------------------------------------------------------

_E2M1 = (0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0)


def _quantize(x, alpha):
    """The quantization rule, whose steps are defined in binary32: (codes 0..15, E4M3 scale bytes)."""
    rows, K = x.shape
    b = x.float().view(rows, K // 16, 16)
    s = (b.abs().amax(2) / (6.0 * alpha)).clamp(max=448.0).to(torch.float8_e4m3fn)
    sigma = s.float()
    r = torch.where(sigma == 0, torch.zeros_like(sigma), 1.0 / (alpha * sigma))
    y = b * r[:, :, None]
    m = y.abs()
    # nearest E2M1 value, a tie goes to the even code
    code = ((m > 0.25).to(torch.uint8) + (m >= 0.75).to(torch.uint8) + (m > 1.25).to(torch.uint8)
            + (m >= 1.75).to(torch.uint8) + (m > 2.5).to(torch.uint8) + (m >= 3.5).to(torch.uint8)
            + (m > 5.0).to(torch.uint8))
    code |= torch.signbit(b).to(torch.uint8) << 3
    return code.view(rows, K), s.view(torch.uint8)


def _alpha(x):
    amax = x.abs().max().float()
    # (a tensor as the divisor: torch multiplies by the reciprocal of a Python number on the GPU)
    return torch.where(amax == 0, torch.ones_like(amax), amax / torch.full_like(amax, 2688.0))


def _values(x, alpha):
    """alpha, and sigma * q of every element in 64 bits."""
    code, sb = _quantize(x, alpha)
    grid = torch.tensor(_E2M1 + tuple(-v for v in _E2M1), dtype=torch.float64, device=x.device)
    sigma = sb.view(torch.float8_e4m3fn).to(torch.float64)
    return grid[code.int()] * sigma.repeat_interleave(16, dim=1)


def _nvfp4_product(x, ax, w):
    aw = _alpha(w)
    return (_values(x, ax) @ _values(w, aw).t()) * (ax.double() * aw.double())


def exact(case, seed):
    t = _tensors(case, seed)
    if case["kind"] == "linear":
        return [_nvfp4_product(x, _alpha(x), w) for x, w in t["pairs"]]
    if case["kind"] == "bf16":
        return [x.double() @ w.double().t() for x, w in t["pairs"]]
    if case["kind"] == "weights":
        w = t["w"]
        N, K = w.shape
        alpha = _alpha(w)
        code, sb = _quantize(w, alpha)
        codes = code[:, 0::2] | (code[:, 1::2] << 4)
        return {"alpha": alpha.view(1).double(), "codes": codes, "scales": sb,
                "kcodes": codes.view(N, K // 64, 32).permute(1, 0, 2).reshape(N, K // 2),
                "kscales": sb.view(N, K // 64, 4).permute(1, 0, 2).reshape(N, K // 16)}
    x = t["x"].double()
    h = (x / torch.sqrt((x * x).mean(1, keepdim=True) + RMS_EPS) * t["norm"].double()).to(torch.bfloat16)
    y1 = _nvfp4_product(h, torch.full((), MLP_ALPHA_IN, device="cuda"), t["w1"])
    gate, up = y1.to(torch.bfloat16).double().chunk(2, dim=1)  # the chain hands on BF16
    p = (gate / (1.0 + torch.exp(-gate)) * up).to(torch.bfloat16)
    y2 = _nvfp4_product(p, torch.full((), MLP_ALPHA_MID, device="cuda"), t["w2"])
    return {"gate_up": y1, "down": y2}
