"""Performance cases of the FlattenQuant linear layer: what a program that serves or prepares a quantized model
calls, over the range of sizes it meets.

Kinds of case (key "kind"):
  linear     the inference call, FqLinear.forward (with "bias": fq_linear_bias): flatten, quantize, integer GEMM,
             dequantize.  "bits" 8, 4 (packed nibbles) or 6 (4-bit values stored as E3M2 codes); "scale" static (the
             calibrated bound, the paper's setting) or dynamic (absmax taken from the activation).
  bmm        fq_bmm_i8 / fq_bmm_i4, the batched product of attention, on operands that are already quantized.
  quantize   fq_flatten_quant_act alone: one activation quantized once for several projections that share it.
  calibrate  fq_channel_absmax with a running maximum: one calibration batch.
  weights    fq_flatten_weights: preparing a layer's weights.

Activations are Gaussian with a share of channels scaled up by log-uniform factors (outlier channels), the channel
maxima come from a calibration batch of 512 rows of the same distribution, and the threshold is three times their
median.  Every result is defined to the bit by the interface, so the tolerance is "exact" throughout.
"""
import math

import numpy as np
import torch

DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
SIZE = {"f32": 4, "f16": 2, "bf16": 2}
DEV = "cuda:0"
MAX_MACS = 16384 * 8192 * 24576          # the largest listed linear layer
MAX_BMM_MACS = 160 * 2048 * 2048 * 128   # four sequences of 40 heads


def listed():
    return [
        # the smallest layer of the test configurations: fp32 in and out, latency only
        dict(name="tiny_i8_f32", kind="linear", M=16, K=256, N=256, bits=8, x="f32", y="f32", scale="dynamic", bias=False,
             outliers=0.016, factor=64.0),
        # decoding one sequence: the attention output projection of a 5120-wide model, calibrated scale
        dict(name="decode1_i8", kind="linear", M=1, K=5120, N=5120, bits=8, x="bf16", y="bf16", scale="static", bias=False,
             outliers=0.01, factor=200.0),
        # decoding a batch of 16 sequences: the up-projection of a 4096-wide model in 4 bits
        dict(name="decode16_i4", kind="linear", M=16, K=4096, N=11008, bits=4, x="bf16", y="bf16", scale="dynamic", bias=False,
             outliers=0.005, factor=100.0),
        # a short prompt (ragged row count) through a biased fp16 layer, as OPT's layers are
        dict(name="prompt77_i8_bias_f16", kind="linear", M=77, K=5120, N=15360, bits=8, x="f16", y="f16", scale="static", bias=True,
             outliers=0.01, factor=200.0),
        # a prompt of 500 tokens, the down-projection in 4 bits
        dict(name="prompt500_i4", kind="linear", M=500, K=11008, N=4096, bits=4, x="bf16", y="bf16", scale="dynamic", bias=False,
             outliers=0.005, factor=100.0),
        # one full context of 2048 tokens through a square INT8 projection
        dict(name="ctx2048_i8", kind="linear", M=2048, K=4096, N=4096, bits=8, x="bf16", y="bf16", scale="dynamic", bias=False,
             outliers=0.005, factor=100.0),
        # batched prefill, 8192 tokens: the 4-bit down-projection, packed nibbles
        dict(name="prefill8192_i4", kind="linear", M=8192, K=11008, N=4096, bits=4, x="bf16", y="bf16", scale="dynamic", bias=False,
             outliers=0.005, factor=100.0),
        # the 4-bit up-projection with its values stored for the 6-bit matrix pipe
        dict(name="prefill8192_e3m2", kind="linear", M=8192, K=4096, N=11008, bits=6, x="bf16", y="bf16", scale="dynamic", bias=False,
             outliers=0.005, factor=100.0),
        # the largest layer of the configurations: 16384 tokens, fused QKV projection of an 8192-wide model
        dict(name="prefill16384_i8", kind="linear", M=16384, K=8192, N=24576, bits=8, x="bf16", y="bf16", scale="static", bias=False,
             outliers=0.003, factor=300.0),
        # attention scores of one 2048-token sequence with 40 heads of 128
        dict(name="attn_qk_i8", kind="bmm", batch=40, M=2048, N=2048, K=128, bits=8, y="bf16"),
        # probabilities times values of the same attention
        dict(name="attn_pv_i8", kind="bmm", batch=40, M=2048, N=128, K=2048, bits=8, y="bf16"),
        # preparing the weights of a 4-bit down-projection
        dict(name="weights_i4", kind="weights", N=5120, K=20480, bits=4, w="bf16", outliers=0.01, factor=200.0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _ragged(rng, v, step, lo):
    """Half of the sizes are multiples of `step`, the others whatever came."""
    return max(lo, v // step * step) if rng.random() < 0.5 else v


def draw(rng):
    kind = rng.choice(["linear"] * 14 + ["bmm"] * 3 + ["quantize", "calibrate", "weights"])
    outl = dict(outliers=rng.choice([0.003, 0.005, 0.01]), factor=rng.choice([64.0, 100.0, 200.0, 300.0]))
    if kind == "linear":
        while True:
            M = _ragged(rng, _log_int(rng, 1, 16384), 64, 1)
            K = _ragged(rng, _log_int(rng, 256, 22016), 128, 256)
            N = _ragged(rng, _log_int(rng, 256, 24576), 128, 256)
            if M * K * N * 1.15 <= MAX_MACS:
                break
        return dict(kind=kind, M=M, K=K, N=N, bits=rng.choice([8, 8, 8, 4, 4, 4, 6]), x=rng.choice(["bf16"] * 4 + ["f16", "f32"]),
                    y=rng.choice(["bf16"] * 4 + ["f16", "f32"]), scale=rng.choice(["static", "dynamic"]),
                    bias=rng.random() < 0.3, **outl)
    if kind == "bmm":
        while True:
            batch, M = rng.choice([1, 8, 12, 32, 40, 64, 96, 160]), _log_int(rng, 1, 2048)
            head, seq = rng.choice([64, 80, 96, 128]), _log_int(rng, 64, 2048)
            N, K = (seq, head) if rng.random() < 0.5 else (head, seq // 32 * 32)
            if batch * M * N * K <= MAX_BMM_MACS:
                break
        return dict(kind=kind, batch=batch, M=M, N=N, K=(K + 31) // 32 * 32, bits=rng.choice([8, 8, 4]), y=rng.choice(["bf16", "bf16", "f16", "f32"]))
    M, K = _log_int(rng, 16, 16384), _ragged(rng, _log_int(rng, 256, 22016), 128, 256)
    if kind == "calibrate":
        return dict(kind=kind, M=M, K=K, x=rng.choice(["bf16", "bf16", "f16", "f32"]), **outl)
    if kind == "weights":
        return dict(kind=kind, N=M, K=K, bits=rng.choice([8, 4, 6]), w=rng.choice(["bf16", "bf16", "f16", "f32"]), **outl)
    return dict(kind=kind, M=M, K=K, bits=rng.choice([8, 4, 6]), x=rng.choice(["bf16", "bf16", "f16", "f32"]),
                scale=rng.choice(["static", "dynamic"]), **outl)


# ------------------------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------------------------
def _rows(buf, K):
    """A [rows, K] view whose rows start on 16-byte boundaries, as the interface asks."""
    return buf[:, :K]


def _normal(g, rows, K, dtype, scale):
    t = torch.randn((rows, (K + 15) // 16 * 16), dtype=torch.float32, device=DEV, generator=g)
    if isinstance(scale, float):
        t *= scale
    else:
        t[:, :K] *= scale
    return _rows(t.to(dtype), K)


def _channels(g, case):
    """Scale of every input channel (1, or an outlier's factor)."""
    K = case["K"]
    n = max(1, int(round(case["outliers"] * K)))
    s = torch.ones(K, dtype=torch.float32, device=DEV)
    at = torch.randperm(K, device=DEV, generator=g)[:n]
    s[at] = torch.exp(torch.rand(n, device=DEV, generator=g) * math.log(case["factor"] / 8.0) + math.log(8.0))
    return s


def _calibration(case, dtype):
    """(channel scales, calibrated channel maxima as numpy fp32, threshold): the model's, whatever the inputs' seed, so
    that the flattened width is the same for all inputs of a case."""
    g = _gen(case["K"])
    s = _channels(g, case)
    chmax = _normal(g, 512, case["K"], dtype, s).float().abs().amax(dim=0).cpu().numpy()
    return s, chmax, float(np.float32(3.0 * np.median(chmax.astype(np.float64))))


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _linear_inputs(case, seed):
    g = _gen(seed)
    dt = DTYPES[case["x"]]
    s, chmax, T = _calibration(case, dt)
    X = _normal(g, case["M"], case["K"], dt, s)
    W = b = None
    if "N" in case:
        W = _normal(g, case["N"], case["K"], torch.bfloat16, 1.0 / math.sqrt(case["K"]))
        b = torch.randn(case["N"], dtype=torch.float32, device=DEV, generator=g) if case["bias"] else None
    return X, W, b, chmax, T


def _bmm_inputs(case, seed):
    """Integer operands (as int8 tensors): attention scores take normal values, a long reduction takes probabilities."""
    g = _gen(seed)
    batch, M, N, K = case["batch"], case["M"], case["N"], case["K"]
    q = 127.0 if case["bits"] == 8 else 7.0
    a = torch.randn((batch, M, K), device=DEV, generator=g)
    if K > 128:
        a = torch.softmax(2.0 * a, dim=2)
    a = torch.round(a * (q / a.abs().max())).to(torch.int8)
    b = torch.randn((batch, N, K), device=DEV, generator=g)
    b = torch.round(b * (q / b.abs().max())).to(torch.int8)
    s = torch.rand(2, device=DEV, generator=g) * 0.02 + 0.005
    return a, b, s


def _nibbles(t):
    return ((t[..., 0::2] & 15) | ((t[..., 1::2] & 15) << 4)).view(torch.uint8)


def _align(bits):
    return 256 if bits == 4 else 128


def _quantized(rows, Kpad, bits):
    if bits == 6:
        return torch.empty((Kpad // 128, rows, 96), dtype=torch.uint8, device=DEV)
    return torch.empty((rows, Kpad if bits == 8 else Kpad // 2), dtype=torch.int8 if bits == 8 else torch.uint8, device=DEV)


def prepare(case, seed):
    import paper_2402_17985_amd as fq
    kind = case["kind"]
    st = dict(case=case, fq=fq)
    if kind == "bmm":
        a, b, s = _bmm_inputs(case, seed)
        if case["bits"] == 4:
            a, b = _nibbles(a), _nibbles(b)
        st.update(a=a, b=b, s_a=s[0:1].clone(), s_b=s[1:2].clone(),
                  Y=torch.empty((case["batch"], case["M"], case["N"]), dtype=DTYPES[case["y"]], device=DEV))
        return st
    if kind == "calibrate":
        g = _gen(seed)
        s = _channels(g, case)
        # the running maximum starts from an earlier batch's
        st.update(X=_normal(g, case["M"], case["K"], DTYPES[case["x"]], s),
                  chmax=_normal(g, 64, case["K"], DTYPES[case["x"]], s).float().abs().amax(dim=0).contiguous())
        return st
    if kind == "weights":
        g = _gen(seed)
        _, chmax, T = _calibration(case, torch.bfloat16)
        W = _normal(g, case["N"], case["K"], DTYPES[case["w"]], 1.0 / math.sqrt(case["K"]))
        src, _, _, Kpad = fq.fq_flatten_plan(chmax, T, _align(case["bits"]))
        st.update(W=W, src=torch.from_numpy(src).to(DEV), Wq=_quantized(case["N"], Kpad, case["bits"]),
                  s_w=torch.empty(1, dtype=torch.float32, device=DEV),
                  ws=torch.empty(fq.fq_weights_workspace_bytes(case["K"], Kpad), dtype=torch.uint8, device=DEV))
        return st
    X, W, b, chmax, T = _linear_inputs(case, seed)
    st["X"] = X
    st["absmax"] = torch.tensor([T], dtype=torch.float32, device=DEV) if case["scale"] == "static" else None
    if kind == "quantize":
        src, rep, _, Kpad = fq.fq_flatten_plan(chmax, T, _align(case["bits"]))
        st.update(src=torch.from_numpy(src).to(DEV), rep=torch.from_numpy(rep).to(DEV), Xq=_quantized(case["M"], Kpad, case["bits"]),
                  s_x=torch.empty(1, dtype=torch.float32, device=DEV),
                  ws=torch.empty(fq.fq_act_workspace_bytes(case["K"], Kpad), dtype=torch.uint8, device=DEV))
        return st
    st["layer"] = fq.FqLinear(W, chmax, T, case["bits"], device=DEV)
    if case["bias"]:
        st["bias"] = b
        st["ws"] = st["layer"].workspace(case["M"])
        st["Y"] = torch.empty((case["M"], case["N"]), dtype=DTYPES[case["y"]], device=DEV)
    return st


def run(st):
    case, fq = st["case"], st["fq"]
    kind = case["kind"]
    if kind == "linear":
        L = st["layer"]
        if case["bias"]:
            fq.fq_linear_bias(st["X"], L.src, L.rep, L.Wq, L.s_w, st["bias"], L.bits, st["Y"], st["ws"], absmax_in=st["absmax"])
            return st["Y"]
        return L.forward(st["X"], out_dtype=DTYPES[case["y"]], absmax_in=st["absmax"])
    if kind == "bmm":
        (fq.fq_bmm_i8 if case["bits"] == 8 else fq.fq_bmm_i4)(st["a"], st["b"], st["s_a"], st["s_b"], st["Y"])
        return st["Y"]
    if kind == "calibrate":
        fq.fq_channel_absmax(st["X"], st["chmax"], accumulate=True)
        return st["chmax"]
    if kind == "weights":
        fq.fq_flatten_weights(st["W"], st["src"], case["bits"], st["Wq"], st["s_w"], st["ws"])
        return st["Wq"], st["s_w"]
    fq.fq_flatten_quant_act(st["X"], st["src"], st["rep"], case["bits"], st["Xq"], st["s_x"], st["ws"], absmax_in=st["absmax"])
    return st["Xq"], st["s_x"]


# ------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ------------------------------------------------------------------------------------------------
QBYTES = {8: 1.0, 4: 0.5, 6: 0.75}


def work(case):
    kind = case["kind"]
    if kind == "bmm":
        b = case["batch"]
        return dict(bytes=b * ((case["M"] + case["N"]) * case["K"] * QBYTES[case["bits"]] + case["M"] * case["N"] * SIZE[case["y"]]),
                    flops=2.0 * b * case["M"] * case["N"] * case["K"])
    if kind == "calibrate":
        return dict(bytes=case["M"] * case["K"] * SIZE[case["x"]] + 8.0 * case["K"], flops=1.0 * case["M"] * case["K"])
    if kind == "weights":
        return dict(bytes=case["N"] * case["K"] * (SIZE[case["w"]] + QBYTES[case["bits"]]), flops=2.0 * case["N"] * case["K"])
    M, K = case["M"], case["K"]
    if kind == "quantize":
        return dict(bytes=M * K * (SIZE[case["x"]] + QBYTES[case["bits"]]), flops=2.0 * M * K)
    # the flattened width is at least K; the quantized activation need not exist in memory
    return dict(bytes=M * K * SIZE[case["x"]] + case["N"] * K * QBYTES[case["bits"]] + M * case["N"] * SIZE[case["y"]],
                flops=2.0 * M * K * case["N"])


def tolerance(case):
    # Integer products are exact, and the interface fixes every rounding around them (scale, dequantized value, output
    # type), so another correct implementation gives the same bits.
    return "exact"


# ------------------------------------------------------------------------------------------------
# the same results in 64 bits
# ------------------------------------------------------------------------------------------------
def exact(case, seed):
    kind = case["kind"]
    if kind == "bmm":
        a, b, s = _bmm_inputs(case, seed)
        out = torch.bmm(a.double(), b.double().transpose(1, 2).contiguous())
        return out * (s[0].double() * s[1].double())
    if kind == "calibrate":
        g = _gen(seed)
        s = _channels(g, case)
        X = _normal(g, case["M"], case["K"], DTYPES[case["x"]], s).abs().amax(dim=0).double()
        return torch.maximum(X, _normal(g, 64, case["K"], DTYPES[case["x"]], s).float().abs().amax(dim=0).double())
    qmax = 127.0 if case["bits"] == 8 else 7.0
    if kind == "weights":
        g = _gen(seed)
        W = _normal(g, case["N"], case["K"], DTYPES[case["w"]], 1.0 / math.sqrt(case["K"]))
        return None, (W.abs().max().double() / qmax).reshape(1)
    X, W, b, chmax, T = _linear_inputs(case, seed)
    # Copies of every channel and the quantized integers, as the interface defines them (scales and multipliers are fp32
    # values, an element is one fp32 product rounded half to even: many products lie on a tie); their product and its
    # scaling then in 64 bits.
    n = torch.from_numpy(np.maximum(1.0, np.ceil(chmax.astype(np.float64) / T))).to(DEV)
    if case["scale"] == "static":
        a = torch.tensor(T, dtype=torch.float64, device=DEV)
    else:
        a = (X.abs().amax(dim=0).double() / n).max().float().double()
    if kind == "quantize":
        return None, (a / qmax).reshape(1)
    qx = torch.clamp(torch.round(X.float() * (qmax / (n * a)).float()), -qmax - 1, qmax).double()
    a_w = W.abs().max().double()
    qw = torch.clamp(torch.round(W.float() * (qmax / a_w).float()), -qmax - 1, qmax).double()
    out = torch.matmul(qx * n, qw.t().contiguous()) * ((a / qmax) * (a_w / qmax))
    return out + b.double() if b is not None else out
