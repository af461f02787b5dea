"""The calls that the library's speed is judged by, over the range of its users' work.

A case is one call of one public entry point on operands that are already on
the GPU: a layer of a network at the size it has in a served or trained model.
`listed()` holds twelve of them, from a 256 x 256 product to an 8192 x 8192
one; `draw()` gives more of the same families and ranges, odd sizes among
them.  Sizes are those of the workloads, tests and documents of this
repository, or generic.
"""
import math

import torch

import paper_2603_06731_amd as pbk

F32, BF16, F16, E4M3, E5M2, INT8 = pbk.PBK_F32, pbk.PBK_BF16, pbk.PBK_F16, pbk.PBK_FP8_E4M3, pbk.PBK_FP8_E5M2, pbk.PBK_INT8
TYPES = {"f32": (F32, torch.float32, 4), "bf16": (BF16, torch.bfloat16, 2), "f16": (F16, torch.float16, 2),
         "e4m3": (E4M3, torch.float8_e4m3fn, 1), "e5m2": (E5M2, torch.float8_e5m2, 1), "int8": (INT8, torch.int8, 1)}
EPILOGUES = {"none": pbk.PBK_EPI_NONE, "bias": pbk.PBK_EPI_BIAS, "relu": pbk.PBK_EPI_RELU, "bias_relu": pbk.PBK_EPI_BIAS_RELU,
             "bias_gelu": pbk.PBK_EPI_BIAS_GELU_TANH, "gelu": pbk.PBK_EPI_GELU_TANH}


# ---------------------------------------------------------------------------- cases

def _matmul(dtype, M, N, K, *, out=None, batch=1, trans_b=0, epi="bias_relu", residual=False):
    return {"kind": "matmul", "dtype": dtype, "out": out or dtype, "batch": batch, "M": M, "N": N, "K": K,
            "trans_b": trans_b, "epi": epi, "residual": residual}


def _conv(dtype, n, H, W, Cin, Cout, k, *, stride=1, pad=0, out=None, epi="bias_relu", transposed=False, residual=False):
    return {"kind": "conv", "dtype": dtype, "out": out or dtype, "n": n, "H": H, "W": W, "Cin": Cin, "Cout": Cout, "k": k,
            "stride": stride, "pad": pad, "epi": epi, "transposed": transposed, "residual": residual}


def _attention(dtype, batch, Nq, Nk, D, *, causal):
    return {"kind": "attention", "dtype": dtype, "batch": batch, "Nq": Nq, "Nk": Nk, "D": D, "causal": causal}


def listed():
    return [
        # the smallest call: a small fp32 layer, where the launch and one chain of latencies are the time
        dict(_matmul("f32", 256, 256, 256), name="matmul_f32_256"),
        # decode: eight tokens through the first matrix of an MLP block (the weights are read once for eight rows)
        dict(_matmul("bf16", 8, 14336, 4096, epi="bias_gelu"), name="matmul_bf16_decode"),
        # an ordinary, ragged size: the second matrix of a vision transformer's MLP for one image of 577 tokens, with the
        # shortcut branch added in the epilogue
        dict(_matmul("bf16", 577, 1024, 4096, epi="bias", residual=True), name="matmul_bf16_block"),
        # the largest product, the headline of the benchmark
        dict(_matmul("bf16", 8192, 8192, 8192), name="matmul_bf16_8192"),
        # the same in FP8 with both operands contiguous along k, as quantised weights are stored
        dict(_matmul("e4m3", 8192, 8192, 8192, out="bf16", trans_b=1), name="matmul_fp8_8192"),
        # attention scores as a batched product: the output is nearly all of the traffic
        dict(_matmul("bf16", 2048, 2048, 128, batch=64, epi="none"), name="scores_bf16"),
        # the 3 x 3 convolution of a residual network's body, at the batch of training or offline inference
        dict(_conv("bf16", 32, 56, 56, 256, 256, 3, pad=1), name="conv_bf16_3x3"),
        # the odd channel count of the paper's worked example: no row of the image is aligned
        dict(_conv("f16", 8, 44, 44, 127, 512, 3, stride=2), name="conv_f16_ragged"),
        # quantised inference: int8 convolution with the batch norm of the layer, int8 codes out
        dict(_conv("int8", 32, 28, 28, 128, 128, 3, pad=1), name="conv_int8_bn"),
        # the upsampling layer of a decoder or generator
        dict(_conv("bf16", 32, 28, 28, 256, 128, 4, stride=2, pad=1, transposed=True), name="conv_transposed_bf16"),
        # prefill: causal self-attention over a prompt
        dict(_attention("bf16", 16, 2048, 2048, 64, causal=True), name="attention_prefill"),
        # decode: one new token attends to a long context
        dict(_attention("bf16", 16, 1, 8192, 128, causal=True), name="attention_decode"),
    ]


def _log(rng, lo, hi):
    """A whole number between lo and hi, evenly over the logarithm."""
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def _size(rng, lo, hi, step, odd=0.25):
    """A size between lo and hi: usually a multiple of `step`, now and then any number."""
    v = _log(rng, lo, hi)
    return v if rng.random() < odd else max(lo, min(hi, v // step * step)) if v >= step else step


def _draw_once(rng):
    f = rng.randrange(12)
    d16 = rng.choice(["bf16", "bf16", "f16"])
    if f == 0:        # small fp32 layers
        return _matmul("f32", _size(rng, 64, 1024, 16), _size(rng, 64, 1024, 16), _size(rng, 64, 1024, 16),
                       trans_b=rng.randrange(2), epi=rng.choice(["bias_relu", "bias", "none"]))
    if f == 1:        # decode: a few rows against a weight matrix
        return _matmul(d16, _log(rng, 1, 64), _size(rng, 1024, 16384, 64), _size(rng, 1024, 16384, 64, odd=0.1),
                       trans_b=rng.randrange(2), epi=rng.choice(["bias_gelu", "bias", "none"]))
    if f == 2:        # the layers of a block for some hundreds or thousands of tokens
        t = rng.randrange(2)
        return _matmul(d16, _size(rng, 128, 4096, 64, odd=0.5), _size(rng, 256, 4096, 64, odd=0.1), _size(rng, 256, 4096, 64, odd=0.1),
                       trans_b=t, epi=rng.choice(["bias", "bias_gelu", "bias_relu"]), residual=rng.random() < 0.5)
    if f == 3:        # large products
        return _matmul(d16, _size(rng, 3072, 8192, 128), _size(rng, 3072, 8192, 128, odd=0.0), _size(rng, 1024, 8192, 128, odd=0.0),
                       trans_b=rng.randrange(2), epi=rng.choice(["bias_relu", "bias_gelu", "none"]))
    if f == 4:        # FP8 products, k-major weights mostly
        return _matmul(rng.choice(["e4m3", "e4m3", "e5m2"]), _size(rng, 64, 8192, 64, odd=0.4), _size(rng, 1024, 8192, 128, odd=0.0),
                       _size(rng, 1024, 8192, 128, odd=0.0), out="bf16", trans_b=int(rng.random() < 0.75),
                       epi=rng.choice(["bias_relu", "bias", "none"]))
    if f == 5:        # scores: batch x heads products with a short contraction
        n = _size(rng, 128, 2048, 64, odd=0.0)
        return _matmul(d16, n, n, rng.choice([32, 64, 64, 128, 128, 256]), batch=_log(rng, 8, 64), trans_b=rng.randrange(2), epi="none")
    if f == 6:        # convolutions of residual networks: 3 x 3 and 1 x 1, stride 1 and 2
        k, s = rng.choice([(3, 1), (3, 1), (3, 2), (1, 1), (1, 2)])
        hw = rng.choice([7, 14, 28, 56])
        return _conv(d16, _log(rng, 1, 64), hw, hw, rng.choice([64, 96, 128, 256, 512]), rng.choice([64, 96, 128, 256, 512]),
                     k, stride=s, pad=k // 2, residual=s == 1 and rng.random() < 0.3)
    if f == 7:        # convolutions with odd channel counts, first layers among them
        hw, k = _log(rng, 14, 224), rng.choice([3, 5, 7])
        return _conv(d16, _log(rng, 1, 8), hw, hw, rng.choice([3, 3, 11, 35, 61, 100, 127]), rng.choice([32, 64, 65, 127, 256, 512]), k,
                     stride=rng.choice([1, 2]), pad=rng.choice([0, k // 2]))
    if f == 8:        # int8 convolutions
        k, hw = rng.choice([1, 3, 3]), rng.choice([7, 14, 28, 56])
        return _conv("int8", _log(rng, 1, 64), hw, hw, rng.choice([32, 64, 128, 256]), rng.choice([32, 64, 128, 256]), k, pad=k // 2,
                     stride=rng.choice([1, 1, 2]))
    if f == 9:        # transposed convolutions: upsampling by two, with and without overlap of the taps
        k = rng.choice([2, 3, 4, 4])
        return _conv(d16, _log(rng, 1, 32), _log(rng, 7, 64), _log(rng, 7, 64), rng.choice([32, 64, 128, 256]),
                     rng.choice([32, 64, 128]), k, stride=2, pad=(k - 1) // 2, transposed=True)
    if f == 10:       # attention of a whole sequence, encoder and decoder
        n = _size(rng, 10, 8192, 64, odd=0.5)
        return _attention(d16, _log(rng, 6, 64), n, n, rng.choice([32, 64, 64, 128, 128]), causal=rng.random() < 0.5)
    # f == 11: decode: one token, or a few, against a context
    return _attention(d16, _log(rng, 16, 256), rng.choice([1, 1, 1, 2, 4, 8]), _log(rng, 128, 8192), rng.choice([64, 128, 128]), causal=True)


def draw(rng):
    while True:
        c = _draw_once(rng)
        w = work(c)
        scale = 0.5 if c["dtype"] in ("e4m3", "e5m2", "int8") else 1.0
        ragged = c["kind"] == "conv" and c["Cin"] % 8
        if w["flops"] * scale <= (1e11 if ragged else 1.1e12) and w["bytes"] <= 6.1e8:
            return c


# ---------------------------------------------------------------------------- sizes and work

def _out_hw(c):
    if c["transposed"]:
        return ((c["H"] - 1) * c["stride"] - 2 * c["pad"] + c["k"], (c["W"] - 1) * c["stride"] - 2 * c["pad"] + c["k"])
    return ((c["H"] + 2 * c["pad"] - c["k"]) // c["stride"] + 1, (c["W"] + 2 * c["pad"] - c["k"]) // c["stride"] + 1)


def work(case):
    c = case
    esz = TYPES[c["dtype"]][2]
    if c["kind"] == "attention":
        pairs, off = c["Nq"] * c["Nk"], c["Nk"] - c["Nq"]
        if c["causal"]:
            pairs = c["Nq"] * off + c["Nq"] * (c["Nq"] + 1) // 2
        return {"bytes": esz * c["batch"] * c["D"] * 2 * (c["Nq"] + c["Nk"]), "flops": 4 * c["batch"] * pairs * c["D"]}
    osz = TYPES[c["out"]][2]
    extra = osz if c["residual"] else 0
    if c["kind"] == "matmul":
        b, M, N, K = c["batch"], c["M"], c["N"], c["K"]
        return {"bytes": esz * b * (M * K + K * N) + (osz + extra) * b * M * N + (4 * N if "bias" in c["epi"] else 0),
                "flops": 2 * b * M * N * K}
    OH, OW = _out_hw(c)
    k2 = c["k"] * c["k"]
    pixels = c["n"] * (c["H"] * c["W"] if c["transposed"] else OH * OW)      # each meets every tap once
    read = c["n"] * (OH * OW if c["k"] == 1 else c["H"] * c["W"])            # a strided 1 x 1 filter skips pixels
    return {"bytes": esz * (read * c["Cin"] + k2 * c["Cin"] * c["Cout"]) + (osz + extra) * c["n"] * OH * OW * c["Cout"]
            + 4 * c["Cout"] * (6 if c["dtype"] == "int8" else 1),
            "flops": 2 * pixels * k2 * c["Cin"] * c["Cout"]}


def tolerance(case):
    # four times the distance of this library's results from the same call worked out in 64 bits
    # int8: integer sums and one binary32 operation per step of the epilogue: the codes are determined
    if case["dtype"] == "int8":
        return "exact"
    # fp32: another order of the sums
    if case["dtype"] == "f32":
        return {"rel": 2e-6, "max": 1.3e-5}
    # attention rounds the weights to 16 bits before they multiply V, then the output once more (the largest
    # differences are in the first rows of a causal prompt, whose few weights do not average)
    if case["kind"] == "attention":
        return {"rel": 9e-3, "max": 0.15} if case["dtype"] == "bf16" else {"rel": 1.2e-3, "max": 1.4e-2}
    # the rest: fp32 sums, rounded once to 16 bits (half a unit in the last place, 2^-9 of the value in bf16)
    return {"rel": 6e-3, "max": 1.6e-2} if case["out"] == "bf16" else {"rel": 8e-4, "max": 2e-3}


# ---------------------------------------------------------------------------- state and pass

class _Inputs:
    """Normal tensors on the GPU, a function of the seed alone."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(self, shape, dtype, std=1.0):
        x = torch.randn(shape, generator=self.g, device="cuda", dtype=torch.float32)
        if std != 1.0:
            x *= std
        if dtype == "int8":
            return x.round_().clamp_(-128, 127).to(torch.int8)
        x = x.to(TYPES[dtype][1])
        return x.view(torch.uint8) if dtype in ("e4m3", "e5m2") else x

    def uniform(self, n, lo, hi):
        return torch.rand(n, generator=self.g, device="cuda", dtype=torch.float32) * (hi - lo) + lo


def prepare(case, seed):
    """The operands, the output buffer and the argument list of the call, as a program with this layer keeps them."""
    c, r = case, _Inputs(seed)
    in_t, out_t = TYPES[c["dtype"]][0], TYPES[c.get("out", c["dtype"])][0]
    stream = torch.cuda.current_stream()

    def empty(*shape):
        return torch.empty(shape, dtype=TYPES[c.get("out", c["dtype"])][1], device="cuda")

    if c["kind"] == "attention":
        b, Nq, Nk, D = c["batch"], c["Nq"], c["Nk"], c["D"]
        q, k, v, o = r.normal((b, Nq, D), c["dtype"]), r.normal((b, Nk, D), c["dtype"]), r.normal((b, Nk, D), c["dtype"]), empty(b, Nq, D)
        dims = (b, Nq, Nk, D, D, D, D, D, Nq * D, Nk * D, Nk * D, Nq * D)
        alpha = 1.0 / math.sqrt(D)
        if c["causal"]:
            return pbk.pbk_attention_causal, (q, k, v, o, *dims, in_t, alpha, stream), o
        return pbk.pbk_attention, (q, k, v, None, o, *dims, 0, 0, in_t, alpha, stream), o

    epi = EPILOGUES[c["epi"]]
    if c["kind"] == "matmul":
        b, M, N, K, t = c["batch"], c["M"], c["N"], c["K"], c["trans_b"]
        A = r.normal((b, M, K), c["dtype"])
        alpha = 1.0
        if c["epi"] == "none":          # a score product: both operands N(0, 1), scaled as scores are
            B, alpha = r.normal((b, N, K) if t else (b, K, N), c["dtype"]), 1.0 / math.sqrt(K)
        else:
            B = r.normal((b, N, K) if t else (b, K, N), c["dtype"], 1.0 / math.sqrt(K))
        bias = r.normal((N,), "f32", 0.1) if "bias" in c["epi"] else None
        C, ldb = empty(b, M, N), K if t else N
        if c["residual"]:
            R = r.normal((M, N), c["out"])
            return pbk.pbk_matmul_residual, (A, B, C, bias, R, M, N, K, K, ldb, N, N, in_t, out_t, t, alpha, 1.0, epi, stream), C
        if b > 1:
            return (pbk.pbk_batched_matmul,
                    (A, B, C, bias, b, M, N, K, K, ldb, N, M * K, K * N, M * N, in_t, out_t, t, alpha, epi, stream), C)
        return pbk.pbk_matmul, (A, B, C, bias, M, N, K, K, ldb, N, in_t, out_t, t, alpha, epi, stream), C

    n, H, W, Cin, Cout, k, s, p = (c[x] for x in ("n", "H", "W", "Cin", "Cout", "k", "stride", "pad"))
    OH, OW = _out_hw(c)
    geometry = (n, H, W, Cin, Cout, k, k, s, s, p, p)
    y = empty(n, OH, OW, Cout)
    if c["dtype"] == "int8":            # codes of activations and weights, and the layer's de-quantisation and batch norm
        x, w = r.normal((n, H, W, Cin), "int8", 40.0), r.normal((k, k, Cin, Cout), "int8", 30.0)
        scale = r.uniform(Cout, 0.5, 2.0) * (3.0 / (40.0 * 30.0 * math.sqrt(k * k * Cin)))
        bias, mean, var = r.normal((Cout,), "f32", 0.5), r.normal((Cout,), "f32", 0.3), r.uniform(Cout, 0.5, 2.0)
        gamma, beta = r.uniform(Cout, 0.5, 1.5), r.normal((Cout,), "f32", 0.3)
        return (pbk.pbk_conv2d_nhwc_int8_bn,
                (x, w, y, *geometry, 1, 1, scale, bias, 0.05, mean, var, 1e-5, gamma, beta, 1, 0.06, out_t, stream), y)
    taps = k * k * Cin / (s * s if c["transposed"] else 1)
    x, w = r.normal((n, H, W, Cin), c["dtype"]), r.normal((k, k, Cin, Cout), c["dtype"], math.sqrt(2.0 / taps))
    bias = r.normal((Cout,), "f32", 0.1)
    if c["transposed"]:
        return pbk.pbk_conv2d_transpose_nhwc, (x, w, y, bias, *geometry, 0, 0, 1, 1, in_t, out_t, 1.0, epi, stream), y
    if c["residual"]:
        R = r.normal((n, OH, OW, Cout), c["out"])
        return pbk.pbk_conv2d_nhwc_residual, (x, w, y, bias, R, *geometry, 1, 1, in_t, out_t, 1.0, 1.0, epi, stream), y
    return pbk.pbk_conv2d_nhwc, (x, w, y, bias, *geometry, 1, 1, in_t, out_t, 1.0, epi, stream), y


def run(state):
    call, args, out = state
    pbk.check(call(*args))
    return out
