"""Performance cases of the FP8-training path: calls a training program makes.

Every case goes through the package's public functions.  A case is a dict of
plain values; ``prepare`` makes its inputs on the GPU (quantized operands,
weights, output buffers and the workspace the library's queries ask for, all
of which a training program allocates once), ``run`` makes one pass over them
and ``work`` says what that pass cannot do without.

Kinds:

* ``gemm``   -- one GEMM with chunk-based FP16 accumulation: ``op`` is
  ``exact`` or ``fast`` (the two modes of FP8 operands), ``sr`` (every
  addition rounded stochastically) or ``p16`` (FP16 operands, the last layer
  of a network).  ``ta``/``tb`` give the direction: Forward (0, 0),
  Backward (0, 1), Gradient (1, 0).  ``fp8out`` also rounds the result back to
  FP8 in the same pass.
* ``update`` -- the weight update with stochastic rounding: ``sgd`` with
  momentum, or ``adam``; both write the FP8 copy for the next step.
* ``conv``   -- one training step of a convolution layer: quantization of the
  input, the implicitly lowered Forward, ReLU, its derivative on the incoming
  error, the Gradient GEMM, the Backward GEMM with col2im, the update.
* ``mlp``    -- one training step of a fully connected network (Fp8Mlp).

All results are codes of the two storage formats (uint8 / uint16), so they are
compared as whole values.
"""
import math

import torch

import paper_1812_08011_amd as fp8t
from paper_1812_08011_amd.mlp import SPEECH_DNN, Fp8Mlp

DEV = "cuda:0"

# Multiply-accumulates of the largest listed case (the conv stage's GEMMs):
# drawn GEMMs stay below it.
MAX_MACS = 50176 * 256 * 2304


def listed():
    return [
        # the smallest call: the unit GEMM of the tests, one small layer
        dict(name="small_exact", kind="gemm", op="exact", ta=0, tb=0, M=128, N=128, K=1024, CL=64,
             data="layer", fp8out=False),
        # a Gradient GEMM whose sizes fit no tile: odd batch, odd widths
        dict(name="ragged_wgrad_exact", kind="gemm", op="exact", ta=1, tb=0, M=1000, N=777, K=3001,
             CL=64, data="layer", fp8out=False),
        # Forward of a 3x3 conv stage (batch 256, 14x14, 256 -> 256), lowered
        dict(name="conv_fwd_exact", kind="gemm", op="exact", ta=0, tb=0, M=50176, N=256, K=2304,
             CL=64, data="layer", fp8out=False),
        # its weight gradient: few outputs, long sums
        dict(name="conv_wgrad_exact", kind="gemm", op="exact", ta=1, tb=0, M=2304, N=256, K=50176,
             CL=64, data="layer", fp8out=False),
        # its Backward GEMM and its weight gradient on the matrix cores
        dict(name="conv_bwd_fast", kind="gemm", op="fast", ta=0, tb=1, M=50176, N=2304, K=256,
             CL=64, data="layer", fp8out=False),
        dict(name="conv_wgrad_fast", kind="gemm", op="fast", ta=1, tb=0, M=2304, N=256, K=50176,
             CL=64, data="layer", fp8out=False),
        # the long-accumulation study: 512 x 512 outputs, 1% outliers
        dict(name="long_sum_exact", kind="gemm", op="exact", ta=1, tb=0, M=512, N=512, K=16384,
             CL=64, data="outliers", fp8out=False),
        # the FP16 last layer of the speech network (batch 256, 1024 -> 6000)
        dict(name="last_layer_p16", kind="gemm", op="p16", ta=0, tb=0, M=256, N=6000, K=1024,
             CL=64, data="layer", fp8out=False),
        # the accumulation study's other rounding mode
        dict(name="long_sum_sr", kind="gemm", op="sr", ta=1, tb=0, M=512, N=512, K=4096, CL=64,
             data="outliers", fp8out=False),
        # the weight update at the parameter count of a 50-layer residual CNN
        dict(name="update_sgd", kind="update", algo="sgd", n=25_600_000, copy8=True),
        # a whole training step of one conv layer at batch 32
        dict(name="conv_layer_step", kind="conv", batch=32, hw=14, cin=256, cout=256, k=3, pad=1,
             stride=1, CL=64),
        # a whole training step of the speech network
        dict(name="speech_step_exact", kind="mlp", mode="exact", batch=256, hidden=1024, layers=6,
             n_in=440, n_out=6000, CL=64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["gemm"] * 5 + ["update", "conv", "mlp"])
    if kind == "update":
        return dict(kind="update", algo=rng.choice(["sgd", "adam"]),
                    n=_log_int(rng, 4096, 25_600_000), copy8=rng.random() < 0.75)
    if kind == "conv":
        k = rng.choice([1, 3, 3, 5])
        return dict(kind="conv", batch=_log_int(rng, 4, 32), hw=rng.choice([7, 14, 15, 28]),
                    cin=rng.choice([32, 48, 64, 100, 128]), cout=rng.choice([32, 64, 96, 128, 130]),
                    k=k, pad=k // 2, stride=rng.choice([1, 1, 2]), CL=64)
    if kind == "mlp":
        return dict(kind="mlp", mode=rng.choice(["exact", "fast"]), batch=_log_int(rng, 32, 256),
                    hidden=rng.choice([256, 500, 768, 1024]), layers=rng.randint(2, 6),
                    n_in=rng.choice([440, 512, 363]), n_out=_log_int(rng, 256, 6000), CL=64)
    op = rng.choice(["exact", "exact", "exact", "fast", "fast", "p16", "sr"])
    ta, tb = rng.choice([(0, 0), (0, 1), (1, 0)])
    # the operations of one multiply-accumulate differ: drawn calls of the
    # variants stay below the largest listed case's time
    cap = MAX_MACS if op in ("exact", "fast") else MAX_MACS // 8
    while True:
        M, N, K = _log_int(rng, 64, 50176), _log_int(rng, 64, 6000), _log_int(rng, 128, 65536)
        if rng.random() < 0.5:            # widths of real layers are multiples of 64
            M, N, K = (max(64, v // 64 * 64) for v in (M, N, K))
        if 128 * 128 * 1024 <= M * N * K <= cap:
            break
    CL = rng.choice([64, 64, 64, 64, 8, 32, 100, 128, 256, K])
    if op in ("p16", "sr"):
        CL = 64
    return dict(kind="gemm", op=op, ta=ta, tb=tb, M=M, N=N, K=K, CL=CL,
                data=rng.choice(["layer", "layer", "outliers"]),
                fp8out=op in ("exact", "fast") and rng.random() < 0.3)


# ---- inputs -------------------------------------------------------------------

def _normal(gen, shape, std=1.0):
    return torch.randn(shape, generator=gen, device=DEV, dtype=torch.float32) * std


def _q8(x, scale=1.0):
    out = torch.empty(x.shape, dtype=torch.uint8, device=DEV)
    return fp8t.fp8_quantize(x, out, scale)


def _q16(x):
    out = torch.empty(x.shape, dtype=torch.uint16, device=DEV)
    return fp8t.fp16_quantize(x, out)


def _outliers(gen, shape):
    z = _normal(gen, shape)
    return torch.where(torch.rand(shape, generator=gen, device=DEV) < 0.01, z * 16.0, z)


def _workspace(nbytes):
    return torch.empty(nbytes, dtype=torch.uint8, device=DEV) if nbytes else None


def _prepare_gemm(c, gen):
    ta, tb, M, N, K = c["ta"], c["tb"], c["M"], c["N"], c["K"]
    a_shape = (K, M) if ta else (M, K)
    b_shape = (N, K) if tb else (K, N)
    a_scale = b_scale = 1.0
    if c["data"] == "outliers":
        a, b = _outliers(gen, a_shape), _outliers(gen, b_shape)
    else:
        # activations (after ReLU) or loss-scaled errors times weights or errors
        if tb:
            a, a_scale = _normal(gen, a_shape, 1e-3), 1024.0
        else:
            a = torch.relu(_normal(gen, a_shape))
        if ta:
            b, b_scale = _normal(gen, b_shape, 1e-3), 1024.0
        else:
            b = _normal(gen, b_shape, math.sqrt(2.0 / K))
    p16 = c["op"] == "p16"
    s = dict(c)
    s["A"] = _q16(a * a_scale) if p16 else _q8(a, a_scale)
    s["B"] = _q16(b * b_scale) if p16 else _q8(b, b_scale)
    s["mode"] = fp8t.FAST if c["op"] == "fast" else fp8t.EXACT
    s["lda"], s["ldb"] = a_shape[1], b_shape[1]
    s["C"] = torch.empty((M, N), dtype=torch.uint16, device=DEV)
    s["out"] = [s["C"].view(torch.int16)]
    args = (ta, tb, M, N, K, c["CL"])
    if c["op"] == "sr":
        s["ws_bytes"] = fp8t.chunk_gemm_sr_workspace_size(*args)
    elif p16:
        s["ws_bytes"] = fp8t.chunk_gemm_p16_workspace_size(*args)
    elif c["fp8out"]:
        s["ws_bytes"] = fp8t.chunk_gemm_fp8_workspace_size(*args, s["mode"])
        s["C8"] = torch.empty((M, N), dtype=torch.uint8, device=DEV)
        s["out"].append(s["C8"])
    else:
        s["ws_bytes"] = fp8t.chunk_gemm_workspace_size(*args, s["mode"])
    s["ws"] = _workspace(s["ws_bytes"])
    s["seed"] = 11
    return s


def _prepare_update(c, gen):
    n = c["n"]
    s = dict(c)
    s["w"] = _q16(_normal(gen, (n,), 0.02))
    s["g"] = _q16(_normal(gen, (n,), 1e-4))
    s["v"] = _q16(_normal(gen, (n,), 1e-4))
    if c["algo"] == "adam":
        s["m"] = _q16(_normal(gen, (n,), 1e-4))
        s["v"] = _q16(_normal(gen, (n,), 1e-4).square())
    s["w8"] = torch.zeros((n,), dtype=torch.uint8, device=DEV) if c["copy8"] else None
    s["t"] = 0
    s["out"] = [s[k].view(torch.int16) for k in ("w", "v", "m") if k in s]
    if c["copy8"]:
        s["out"].append(s["w8"])
    return s


def _conv_sizes(c):
    o = (c["hw"] + 2 * c["pad"] - c["k"]) // c["stride"] + 1
    return o, c["batch"] * o * o, c["k"] * c["k"] * c["cin"]


def _prepare_conv(c, gen):
    o, M, K = _conv_sizes(c)
    cin, cout, CL, B, hw = c["cin"], c["cout"], c["CL"], c["batch"], c["hw"]
    u8 = lambda *shape: torch.empty(shape, dtype=torch.uint8, device=DEV)
    u16 = lambda *shape: torch.empty(shape, dtype=torch.uint16, device=DEV)
    s = dict(c, o=o, M=M, K=K)
    s["X"] = torch.relu(_normal(gen, (B, hw, hw, cin)))
    s["D16"] = _q16(_normal(gen, (M, cout), 1e-3 * 1024.0))
    s["W16"] = _q16(_normal(gen, (K, cout), math.sqrt(2.0 / K)))
    s["W8"] = u8(K, cout)
    fp8t.fp8_quantize(s["W16"], s["W8"])
    s["V16"] = torch.zeros((K, cout), dtype=torch.int16, device=DEV).view(torch.uint16)
    s["X8"], s["Y16"], s["Y8"], s["A8"] = u8(B, hw, hw, cin), u16(M, cout), u8(M, cout), u8(M, cout)
    s["E8"], s["dW"], s["dcol"], s["dX"] = u8(M, cout), u16(K, cout), u16(M, K), u16(B, hw, hw, cin)
    conv = (B, hw, hw, cin, c["k"], c["k"], c["pad"], c["stride"])
    s["conv"] = conv
    s["ws_bytes"] = max(fp8t.conv2d_workspace_size(0, *conv, cout, CL),
                        fp8t.conv2d_workspace_size(1, *conv, cout, CL),
                        fp8t.chunk_gemm_workspace_size(0, 1, M, K, cout, CL, fp8t.EXACT))
    s["ws"] = _workspace(s["ws_bytes"])
    s["t"] = 0
    s["out"] = dict(A8=s["A8"], Y16=s["Y16"].view(torch.int16), dW=s["dW"].view(torch.int16),
                    dX=s["dX"].view(torch.int16), W16=s["W16"].view(torch.int16), W8=s["W8"])
    return s


def _widths(c):
    if (c["n_in"], c["n_out"], c["hidden"], c["layers"]) == (440, 6000, 1024, 6):
        return SPEECH_DNN
    return (c["n_in"],) + (c["hidden"],) * (c["layers"] - 1) + (c["n_out"],)


def _prepare_mlp(c, gen):
    w = _widths(c)
    net = Fp8Mlp(w, c["batch"], c["CL"], fp8t.FAST if c["mode"] == "fast" else fp8t.EXACT, DEV)
    for l in range(net.L):
        fp8t.fp16_quantize(_normal(gen, (w[l], w[l + 1]), 1.0 / math.sqrt(w[l])), net.W16[l])
        if l < net.L - 1:
            fp8t.fp8_quantize(net.W16[l], net.W8[l])
    s = dict(c, net=net, t=0)
    s["X8"] = _q8(_normal(gen, (c["batch"], w[0])))
    s["T16"] = _q16(_normal(gen, (c["batch"], w[-1])))
    view = lambda ts: [t.view(torch.int16) for t in ts]
    s["out"] = dict(Y=net.Y16.view(torch.int16), W=view(net.W16), V=view(net.V16),
                    dW=view(net.dW16), W8=net.W8)
    return s


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    return {"gemm": _prepare_gemm, "update": _prepare_update, "conv": _prepare_conv,
            "mlp": _prepare_mlp}[case["kind"]](case, gen)


# ---- one pass -------------------------------------------------------------------

def _run_gemm(s):
    args = (s["ta"], s["tb"], s["M"], s["N"], s["K"], s["CL"], s["A"], s["lda"], s["B"], s["ldb"],
            s["C"], s["N"])
    if s["op"] == "sr":
        fp8t.chunk_gemm_sr(*args, s["seed"], 0, s["ws"], s["ws_bytes"])
    elif s["op"] == "p16":
        fp8t.chunk_gemm_p16(*args, s["ws"], s["ws_bytes"])
    elif s["fp8out"]:
        fp8t.chunk_gemm_fp8(*args, s["C8"], s["N"], 1.0, s["mode"], s["ws"], s["ws_bytes"])
    else:
        fp8t.chunk_gemm(*args, s["mode"], s["ws"], s["ws_bytes"])
    return s["out"]


def _run_update(s):
    s["t"] += 1
    if s["algo"] == "sgd":
        fp8t.sr_weight_update(s["w"], s["g"], s["v"], s["w8"], s["n"], 0.1, 0.9, 1e-4, 7, s["t"])
    else:
        fp8t.adam_update(s["w"], s["g"], s["m"], s["v"], s["w8"], s["n"], 1e-3, 0.9, 0.999, 1e-8,
                         1e-4, s["t"], 7, s["t"])
    return s["out"]


def _run_conv(s):
    conv, M, K, cout, CL = s["conv"], s["M"], s["K"], s["cout"], s["CL"]
    ws = (s["ws"], s["ws_bytes"])
    fp8t.fp8_quantize(s["X"], s["X8"])
    fp8t.conv2d_fwd_fp8(s["X8"], *conv, s["W8"], cout, CL, s["Y16"], cout, *ws)
    fp8t.fp8_quantize(s["Y16"], s["Y8"])
    fp8t.relu_codes(s["Y8"], 8, s["A8"], M * cout)
    fp8t.relu_backward_fp8(s["D16"], s["Y16"], s["E8"], M * cout)
    fp8t.conv2d_wgrad_fp8(s["X8"], *conv, s["E8"], cout, CL, s["dW"], cout, *ws)
    fp8t.chunk_gemm(0, 1, M, K, cout, CL, s["E8"], cout, s["W8"], cout, s["dcol"], K, fp8t.EXACT,
                    *ws)
    fp8t.col2im_fp16(s["dcol"], *conv, s["dX"])
    s["t"] += 1
    # lr / loss scale, weight decay x loss scale: the gradients carry the scale
    fp8t.sr_weight_update(s["W16"], s["dW"], s["V16"], s["W8"], K * cout, 1e-5 / 1024.0, 0.9,
                          1e-4 * 1024.0, 7, s["t"])
    return s["out"]


def _run_mlp(s):
    s["t"] += 1
    s["net"].step(s["X8"], s["T16"], 0.003, 0.9, 1e-4, 1000.0, 21, s["t"])
    return s["out"]


def run(state):
    return {"gemm": _run_gemm, "update": _run_update, "conv": _run_conv,
            "mlp": _run_mlp}[state["kind"]](state)


# ---- what a pass cannot do without -------------------------------------------------

def work(case):
    c = case
    if c["kind"] == "gemm":
        M, N, K = c["M"], c["N"], c["K"]
        eb = 2 if c["op"] == "p16" else 1
        return {"bytes": eb * (M * K + K * N) + (3 if c["fp8out"] else 2) * M * N,
                "flops": 2 * M * N * K}
    if c["kind"] == "update":
        # w, g, v (adam: m, too) in; w, v (m) out; the FP8 copy
        n, adam = c["n"], c["algo"] == "adam"
        return {"bytes": n * ((14 if adam else 10) + (1 if c["copy8"] else 0)),
                "flops": n * (16 if adam else 6)}
    if c["kind"] == "conv":
        _, M, K = _conv_sizes(c)
        x, cout = c["batch"] * c["hw"] ** 2 * c["cin"], c["cout"]
        # input in, dX out; Y, D, A8 of the outputs; weights, momentum, copy
        return {"bytes": x * (4 + 2) + M * cout * (2 + 2 + 1) + K * cout * (2 * 4 + 2),
                "flops": 3 * 2 * M * K * cout}
    w, B = _widths(c), c["batch"]
    params = [w[l] * w[l + 1] for l in range(len(w) - 1)]
    macs = sum((3 if l else 2) * B * p for l, p in enumerate(params))
    # per parameter: w, v read and written, dw written, the FP8 copy read and
    # written; the input, the logits and the targets
    return {"bytes": 12 * sum(params) + B * (w[0] + 4 * w[-1]), "flops": 2 * macs}


def tolerance(case):
    # Exact mode, SR, FP16 operands and the updates are defined bit for bit.
    # Fast mode leaves the order of the products inside a chunk open; measured
    # over its five matrix-core kernels (16x16x32, 32x32x16 and 32x32x64
    # instructions) on layer data and on data with outliers, CL 64, 128, 256
    # and 2496, no code differed.
    return "exact"


def exact(case, seed):
    """None: every output is a code of the FP8 or FP16 storage format (a whole
    number), with each addition's rounding part of its definition."""
    return None
