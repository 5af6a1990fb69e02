"""Timed workloads of the W4Ax path: what a serving program asks of this library.

Each case is one step of a LLaMA-3-shaped model through the public binding, with
synthetic inputs made on the GPU from a seed:

  linear   quantize the fp16 activations, then the W4Ax GEMM (optionally with
           the calibrated channel permutation in the quantizer)
  mlp      quantize, gate/up GEMM with SwiGLU and the next quantization fused,
           then the down GEMM
  kv4_q    4-bit quantization of K or V rows as they enter the cache
  kv4_dq   the inverse, for a reader of the cache

Activations are N(0, 1) with the channels of the 8-bit blocks (or, for
calibrated layers, 0.5% of the channels, scattered) 50 times larger; weights are
N(0, 0.02^2); K/V rows have per-channel ranges 2^U(0, 3).
"""
import math

import numpy as np
import torch

import paper_2410_12168_amd as comet

G = 128
# (K, N) of the LLaMA-3 layers
SHAPES = {
    "8b": {"qkv": (4096, 6144), "o": (4096, 4096), "gate_up": (4096, 28672), "down": (14336, 4096)},
    "70b": {"qkv": (8192, 10240), "o": (8192, 8192), "gate_up": (8192, 57344),
            "down": (28672, 8192)},
}


def _linear(name, M, model, layer, frac8=0.0625, placement="contiguous", perm=False):
    K, N = SHAPES[model][layer]
    return {"name": name, "kind": "linear", "M": M, "K": K, "N": N, "frac8": frac8,
            "placement": placement, "perm": perm}


def listed():
    return [
        # the smallest layer in use: latency of two dependent launches
        {"name": "tiny_linear_m16", "kind": "linear", "M": 16, "K": 1024, "N": 1024,
         "frac8": 0.125, "placement": "contiguous", "perm": False},
        # one user's token: the small layer of the small model
        _linear("decode_8b_qkv_m1", 1, "8b", "qkv"),
        # a few users' tokens: the layer with most of the weights
        _linear("decode_70b_gate_up_m8", 8, "70b", "gate_up"),
        # a serving batch over the long-K layer, 8-bit blocks scattered
        _linear("decode_70b_down_m48", 48, "70b", "down", placement="random"),
        # a large serving batch
        _linear("batch_70b_gate_up_m128", 128, "70b", "gate_up"),
        # a short prompt or a chunk of one, ragged
        _linear("chunk_70b_down_m333", 333, "70b", "down"),
        # a ragged prefill of the small model, no 8-bit block
        _linear("prefill_8b_o_m1900", 1900, "8b", "o", frac8=0.0),
        # prefill with the calibrated permutation
        _linear("prefill_70b_qkv_m4096_perm", 4096, "70b", "qkv", perm=True),
        # a whole MLP on a mid-sized prompt
        {"name": "mlp_8b_m512", "kind": "mlp", "M": 512, "K": 4096, "I": 14336, "frac8": 0.0625,
         "placement": "contiguous"},
        # the dominant layer of a long prefill
        _linear("prefill_70b_gate_up_m4096", 4096, "70b", "gate_up"),
        # K or V of one layer of a prefill batch of 8 x 4096 tokens into the cache
        {"name": "kv4_quantize_t32768", "kind": "kv4_q", "T": 32768, "C": 1024, "G": 128},
        # a reader of the cache: ragged length, the finest groups
        {"name": "kv4_dequantize_t20001", "kind": "kv4_dq", "T": 20001, "C": 1024, "G": 32},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["linear"] * 7 + ["mlp"] * 2 + ["kv4_q", "kv4_dq"])
    if kind.startswith("kv4"):
        return {"kind": kind, "T": _log(rng, 1, 32768), "C": rng.choice([512, 1024, 2048]),
                "G": rng.choice([32, 64, 128])}
    M = _log(rng, 1, 4096)
    frac8 = rng.choice([0.0, 0.0625, 0.0625, 0.0625, 0.25, 0.5])
    placement = rng.choice(["contiguous", "random"])
    if kind == "mlp":
        K = 128 * _log(rng, 8, 64)
        I = 128 * _log(rng, 16, 112)
        return {"kind": "mlp", "M": M, "K": K, "I": I, "frac8": frac8, "placement": placement}
    if rng.random() < 0.5:  # a layer of the models, else any size between them
        K, N = rng.choice([s for m in SHAPES.values() for s in m.values()])
    else:
        K, N = 128 * _log(rng, 8, 224), 16 * _log(rng, 64, 3584)
        while K * N > 8192 * 57344:
            N = max(16, N // 32 * 16)
    perm = rng.random() < 0.2
    return {"kind": "linear", "M": M, "K": K, "N": N, "frac8": frac8, "placement": placement,
            "perm": perm}


def _prec(K, frac8, placement, seed):
    """Block precisions: a run of 8-bit blocks from block 3 NG / 8, or a random subset."""
    NG = K // G
    m = np.full(NG, 4, np.uint8)
    n8 = int(round(frac8 * NG))
    if placement == "random":
        m[np.random.default_rng(seed).permutation(NG)[:n8]] = 8
    else:
        m[(3 * NG // 8 + np.arange(n8)) % NG] = 8
    return m


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _normal(g, rows, cols, std=1.0):
    """fp16 [rows][cols]; made in slices, so that fp32 copies stay small."""
    out = torch.empty((rows, cols), dtype=torch.float16, device="cuda")
    step = max(1, (1 << 27) // cols)
    for r in range(0, rows, step):
        n = min(step, rows - r)
        out[r:r + n] = torch.randn((n, cols), generator=g, device="cuda").mul_(std)
    return out


def _inputs(case, seed):
    """The tensors a case starts from, and its host maps."""
    g = _gen(seed)
    kind = case["kind"]
    if kind.startswith("kv4"):
        T, C = case["T"], case["C"]
        x = torch.randn((T, C), generator=g, device="cuda")
        x *= torch.exp2(3.0 * torch.rand(C, generator=g, device="cuda"))
        return {"x": x.half()}
    M, K = case["M"], case["K"]
    N = 2 * case["I"] if kind == "mlp" else case["N"]
    x = _normal(g, M, K)
    w = _normal(g, N, K, 0.02)
    if case.get("perm"):
        chan = torch.randperm(K, generator=g, device="cuda")[:max(1, K // 200)]
        x[:, chan] *= 50.0
        absmax = x[:512].abs().amax(dim=0).float()
        perm, prec, _ = comet.plan_channel_perm(absmax)
        return {"x": x, "w": w, "prec": prec, "perm": torch.from_numpy(perm).cuda()}
    prec = _prec(K, case["frac8"], case["placement"], seed)
    x *= torch.from_numpy(np.repeat(np.where(prec == 8, 50.0, 1.0), G)).half().cuda()
    out = {"x": x, "w": w, "prec": prec, "perm": None}
    if kind == "mlp":
        out["w2"] = _normal(g, K, case["I"], 0.02)
        out["prec2"] = _prec(case["I"], case["frac8"], case["placement"], seed + 1)
    return out


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case, **_inputs(case, seed)}
    if kind == "kv4_q":
        return s
    if kind == "kv4_dq":
        s["codes"], s["params"] = comet.kv4_quantize(s.pop("x"), case["G"])
        return s
    M, K = case["M"], case["K"]
    w = s.pop("w")
    s["N"] = N = w.shape[0]
    s["W"], s["sw"] = comet.pack_w4(w, s["perm"])
    # a serving program's buffers, kept between calls
    s["A"] = torch.empty(comet.comet_act_packed_bytes(s["prec"], M, K), dtype=torch.uint8,
                         device="cuda")
    s["sa"] = torch.empty((K // G, M), dtype=torch.float16, device="cuda")
    if kind == "mlp":
        I = case["I"]
        s["W2"], s["sw2"] = comet.pack_w4(s.pop("w2"))
        s["A2"] = torch.empty(comet.comet_act_packed_bytes(s["prec2"], M, I), dtype=torch.uint8,
                              device="cuda")
        s["sa2"] = torch.empty((I // G, M), dtype=torch.float16, device="cuda")
        s["out"] = torch.empty((M, K), dtype=torch.float16, device="cuda")
    else:
        s["out"] = torch.empty((M, N), dtype=torch.float16, device="cuda")
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "kv4_q":
        return comet.kv4_quantize(s["x"], case["G"])
    if kind == "kv4_dq":
        return comet.kv4_dequantize(s["codes"], s["params"], case["G"])
    M, K, N = case["M"], case["K"], s["N"]
    if s["perm"] is None:
        comet.comet_fmpq_quantize_act(s["x"], s["prec"], s["A"], s["sa"], M, K)
    else:
        comet.comet_fmpq_quantize_act_perm(s["x"], s["perm"], s["prec"], s["A"], s["sa"], M, K)
    if kind == "linear":
        comet.comet_w4ax_gemm(s["A"], s["prec"], s["sa"], s["W"], s["sw"], s["out"], M, N, K)
        return s["out"]
    comet.comet_w4ax_gemm_swiglu_quant(s["A"], s["prec"], s["sa"], s["W"], s["sw"], M, N, K, G,
                                       s["prec2"], s["A2"], s["sa2"])
    comet.comet_w4ax_gemm(s["A2"], s["prec2"], s["sa2"], s["W2"], s["sw2"], s["out"], M, K,
                          case["I"])
    return s["out"]


def work(case):
    if case["kind"].startswith("kv4"):
        T, C, g = case["T"], case["C"], case["G"]
        return {"bytes": 2 * T * C + T * C // 2 + 4 * T * (C // g), "flops": 0}
    M, K = case["M"], case["K"]
    if case["kind"] == "mlp":
        I = case["I"]
        w = 3 * I * K // 2 + 2 * 3 * I * K // G
        return {"bytes": 4 * M * K + w, "flops": 6 * M * I * K}
    N = case["N"]
    return {"bytes": 2 * M * K + N * K // 2 + 2 * N * K // G + 2 * M * N, "flops": 2 * M * N * K}


def tolerance(case):
    # Codes and parameters of the KV cache, and the values they stand for, are
    # defined bit by bit.
    if case["kind"].startswith("kv4"):
        return "exact"
    # Between the two GEMMs of the MLP a value on a rounding edge of the 4-bit
    # quantizer may take the neighbouring code.
    if case["kind"] == "mlp":
        return {"rel": 1e-2}
    # fp32 sums rounded once to fp16: 2e-4 in the 2-norm, at most one fp16 step
    # (2^-10 of the value) in one element.
    return {"rel": 8e-4, "max": 2e-3}


def _fake_quant(x, prec):
    """fp16 [R][K] -> the fp64 values that its codes and scales stand for."""
    R, K = x.shape
    b = x.float().view(R, K // G, G)
    qmax = torch.from_numpy(np.where(np.asarray(prec) == 8, 127.0, 7.0)).float().to(x.device)
    qmax = qmax.view(1, -1, 1)
    sc = (b.abs().amax(dim=2, keepdim=True) / qmax).half().float()
    q = torch.where(sc > 0, torch.round(b / torch.where(sc > 0, sc, 1.0)), 0.0)
    q = torch.minimum(torch.maximum(q, -qmax), qmax)
    return (q.double() * sc.double()).view(R, K)


def _product(a, w):
    """a (fp64 [M][K]) times the quantized w (fp16 [N][K]) transposed, in slices of N."""
    N, K = w.shape
    four = np.full(K // G, 4, np.uint8)
    out = torch.empty((a.shape[0], N), dtype=torch.float64, device=a.device)
    step = max(16, (1 << 27) // K)
    for n in range(0, N, step):
        out[:, n:n + step] = a @ _fake_quant(w[n:n + step], four).t()
    return out


def exact(case, seed):
    if case["kind"].startswith("kv4"):
        return None
    s = _inputs(case, seed)
    x, w = s["x"], s["w"]
    if s["perm"] is not None:
        x, w = x[:, s["perm"].long()], w[:, s["perm"].long()]
    y = _product(_fake_quant(x, s["prec"]), w)
    if case["kind"] == "linear":
        return y
    # gate and up columns alternate in groups of 128; h is kept in fp16
    M, I = case["M"], case["I"]
    y = y.half().double().view(M, I // G, 2, G)
    h = (y[:, :, 0] * torch.sigmoid(y[:, :, 0]) * y[:, :, 1]).reshape(M, I).half()
    return _product(_fake_quant(h, s["prec2"]), s["w2"])
