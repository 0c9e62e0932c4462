"""The calls this library is used for, at the sizes it is used at.

Each case is one pass through the public entry points of
``paper_2311_14114_amd``, on inputs drawn on the GPU from a seed.  The kinds:

  linear   one quantized linear layer, ``soniq_quantize_mp_gemm`` into a
           caller's output: decode rows, short prompts, full batches
  conv     one 3x3 convolution from its NCHW input through the haloed code
           image (``soniq_quantize_act_conv3x3`` + ``soniq_mp_gemm``)
  ffn      two linear layers, the second one's input quantized by the first
           one's kernel, with its batch maximum or with calibrated scales
  stack    a decode step: the linear layers of several decoder blocks,
           captured once in a HIP graph and replayed per token, as a serving
           loop runs them (every layer has weights of its own, so they come
           from HBM and not from a cache)

Activations are N(0,1) (|N(0,1)| after a ReLU, for unsigned layers); with
``outliers`` the wide channels are 20 times larger, as in transformer
encoders.  Weights are N(0, 0.02), filters N(0, 0.05).  Which channels are
narrow is a random choice per seed, never sorted.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2311_14114_amd as sq


def _linear(name, M, N, K, *, a=(4, 8), a_lo_share=0.5, w=(2, 4), w_lo_share=0.75, a_signed=True,
            outliers=False, group_bits=0, dense=False):
    return dict(name=name, kind="linear", M=M, N=N, K=K, a_lo=a[0], a_hi=a[1], a_lo_share=a_lo_share,
                w_lo=w[0], w_hi=w[1], w_lo_share=w_lo_share, a_signed=a_signed, outliers=outliers,
                group_bits=group_bits, dense=dense)


def _decode(name, M, N, K, **more):
    return _linear(name, M, N, K, a_lo_share=0.8, **more)


def _encoder(name, M, N, K, **more):
    return _linear(name, M, N, K, a_lo_share=0.99, w=(2, 8), w_lo_share=0.7, outliers=True, **more)


def listed():
    return [
        # the smallest layer of the test set: what a call costs when the work is nothing
        _linear("tiny_linear", 64, 256, 256),
        # one token through the up projection of a 4096-wide decoder, one call
        _decode("decode_m1", 1, 11008, 4096),
        # eight sequences decoded together through the same layer
        _decode("decode_m8", 8, 11008, 4096),
        # the same batch with 3- and 6-bit weights, stored at their own width
        _decode("decode_m8_w36_dense", 8, 11008, 4096, w=(3, 6), dense=True),
        # the same batch with one activation scale per 512 bits of channels
        _decode("decode_m8_g512", 8, 11008, 4096, group_bits=512),
        # a decode step at one sequence: six blocks' projections and FFNs in a graph
        dict(name="decode_stack_m1", kind="stack", M=1, K=4096, F=11008, layers=6),
        # a short prompt of an odd length against odd widths, unsigned activations
        _linear("ragged_prompt", 301, 4099, 4091, a_lo_share=0.8, w=(3, 6), a_signed=False),
        # ResNet-18's 256-channel 3x3 convolution at 14x14, batch 32
        dict(name="conv3x3_resnet", kind="conv", B=32, C=256, H=14, W=14, N=256),
        # encoder layers, hidden 768, 128 tokens x batch 32
        _encoder("encoder_qkv", 4096, 2304, 768),
        dict(name="encoder_ffn", kind="ffn", M=4096, K=768, F=3072, N=768, static=False),
        _encoder("encoder_ffn_down_g512", 4096, 768, 3072, group_bits=512),
        # the largest product: 8192 cubed, half of the channels wide on both sides
        _linear("square_8192", 8192, 8192, 8192, w=(4, 8), w_lo_share=0.5),
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["decode", "decode", "linear", "linear", "encoder", "grouped", "conv", "ffn", "stack"])
    widths = rng.choice([(2, 4), (2, 8), (4, 8), (3, 6)])
    if kind == "decode":
        c = _decode("", rng.randint(1, 8), size(1024, 16384), size(1024, 12288), w=widths,
                    dense=rng.random() < 0.3)
    elif kind == "linear":
        c = _linear("", size(9, 8192), size(200, 8192), size(200, 8192), w=widths,
                    a_lo_share=rng.choice([0.5, 0.8]), a_signed=rng.random() < 0.7)
    elif kind == "encoder":
        c = _encoder("", size(256, 8192), 64 * rng.randint(8, 64), 64 * rng.randint(8, 64))
    elif kind == "grouped":
        c = _linear("", size(1, 4096), size(512, 8192), 4 * size(128, 2048), w=widths, a_lo_share=0.8,
                    group_bits=512)
    elif kind == "conv":
        hw = rng.randint(7, 56)
        c = dict(kind="conv", B=rng.randint(1, 32), C=16 * rng.randint(2, 16), H=hw,
                 W=max(7, hw + rng.randint(-2, 2)), N=16 * rng.randint(2, 16))
    elif kind == "ffn":
        k = 64 * rng.randint(6, 32)
        c = dict(kind="ffn", M=size(1, 8192), K=k, F=4 * k, N=k, static=rng.random() < 0.5)
    else:
        k = 64 * rng.randint(16, 64)
        c = dict(kind="stack", M=rng.randint(1, 8), K=k, F=64 * round(k * 8 / 3 / 64),
                 layers=rng.randint(2, 6))
    c.pop("name", None)
    return c


# ------------------------------------------------------------------ inputs

def _split(rng, n, lo_share, lo, hi):
    bits = np.full(n, hi, np.uint8)
    bits[rng.permutation(n)[:int(round(lo_share * n))]] = lo
    return bits


class _Draw:
    """One case's random numbers: tensors on the GPU, channel widths on the host."""

    def __init__(self, seed):
        self.host = np.random.Generator(np.random.PCG64(seed))
        self.dev = torch.Generator(device="cuda")
        self.dev.manual_seed(seed)

    def normal(self, *shape):
        return torch.randn(*shape, device="cuda", dtype=torch.float32, generator=self.dev)


def _layer(d, N, K, a_bits, w=(2, 4), w_lo_share=0.75):
    return dict(W=d.normal(N, K).mul_(0.02), a_bits=a_bits, w_bits=_split(d.host, N, w_lo_share, *w))


def _encoder_layer(d, N, K):
    return _layer(d, N, K, _split(d.host, K, 0.99, 4, 8), (2, 8), 0.7)


def _decode_layer(d, N, K):
    return _layer(d, N, K, _split(d.host, K, 0.8, 4, 8))


def _outliers(A, a_bits):
    A[:, torch.from_numpy(np.flatnonzero(a_bits == a_bits.max())).cuda()] *= 20.0
    return A


def _static_scales(a_bits, std):
    """Calibrated scales of a layer's input: 4.5 standard deviations at the top code."""
    return [4.5 * std / (2 ** (int(b) - 1) - 1) for b in sorted(set(a_bits.tolist()))]


def _data(case, seed):
    """The case's matrices and widths, before any packing."""
    d = _Draw(seed)
    kind = case["kind"]
    if kind == "linear":
        a_bits = _split(d.host, case["K"], case["a_lo_share"], case["a_lo"], case["a_hi"])
        A = d.normal(case["M"], case["K"])
        if not case["a_signed"]:
            A.abs_()
        if case["outliers"]:
            _outliers(A, a_bits)
        return dict(A=A, layer=_layer(d, case["N"], case["K"], a_bits, (case["w_lo"], case["w_hi"]),
                                      case["w_lo_share"]))
    if kind == "conv":
        C, N = case["C"], case["N"]
        X = d.normal(case["B"], C, case["H"], case["W"]).abs_()
        F = d.normal(N, C, 3, 3).mul_(0.05)
        return dict(X=X, F=F, c_bits=_split(d.host, C, 0.6, 4, 8), w_bits=_split(d.host, N, 0.8, 1, 4))
    if kind == "ffn":
        up = _encoder_layer(d, case["F"], case["K"])
        down = _encoder_layer(d, case["N"], case["F"])
        A = _outliers(d.normal(case["M"], case["K"]), up["a_bits"])
        n_wide = int((up["a_bits"] == 8).sum())
        std = 0.02 * math.sqrt(case["K"] + 399 * n_wide)
        return dict(A=A, up=up, down=down, s_next=_static_scales(down["a_bits"], std))
    M, K, F = case["M"], case["K"], case["F"]
    blocks = []
    for _ in range(case["layers"]):
        o, up, down = _decode_layer(d, K, K), _decode_layer(d, F, K), _decode_layer(d, K, F)
        blocks.append(dict(o=o, up=up, down=down, x_o=d.normal(M, K), x_f=d.normal(M, K),
                           s_next=_static_scales(down["a_bits"], 0.02 * math.sqrt(K))))
    return dict(blocks=blocks)


def _pack(layer, a_signed=True, **more):
    return sq.soniq_pack_weights(layer["W"], layer["w_bits"], layer["a_bits"], a_signed, **more)


def _out(M, N):
    return torch.empty((M, N), dtype=torch.bfloat16, device="cuda")


def prepare(case, seed):
    data = _data(case, seed)
    kind = case["kind"]
    if kind == "linear":
        w = _pack(data["layer"], case["a_signed"], act_group_bits=case["group_bits"], dense=case["dense"])
        return dict(kind=kind, w=w, act=sq.soniq_act_create(w, case["M"]), A=data["A"],
                    Y=_out(case["M"], case["N"]))
    if kind == "conv":
        w = sq.soniq_pack_weights_conv3x3(data["F"], data["w_bits"], data["c_bits"], False, sign_nibbles=True)
        act = sq.soniq_act_create_conv3x3(w, case["B"], case["H"], case["W"])
        return dict(kind=kind, w=w, act=act, X=data["X"], Y=_out(act.max_M, case["N"]))
    if kind == "ffn":
        M = case["M"]
        up, down = _pack(data["up"]), _pack(data["down"])
        return dict(kind=kind, static=case["static"], up=up, down=down, A=data["A"],
                    s_next=np.asarray(data["s_next"], np.float32), act_up=sq.soniq_act_create(up, M),
                    act_down=sq.soniq_act_create(down, M), H=_out(M, case["F"]), Y=_out(M, case["N"]))
    M = case["M"]
    blocks = []
    for b in data["blocks"]:
        s = dict(x_o=b["x_o"], x_f=b["x_f"], s_next=np.asarray(b["s_next"], np.float32))
        for n in ("o", "up", "down"):
            s[n] = _pack(b[n])
            s["act_" + n] = sq.soniq_act_create(s[n], M)
        s["Y_o"], s["Y"] = _out(M, case["K"]), _out(M, case["K"])
        blocks.append(s)

    def step():
        for s in blocks:
            sq.soniq_quantize_mp_gemm(s["act_o"], s["o"], s["x_o"], out=s["Y_o"])
            sq.soniq_quantize_act(s["act_up"], s["x_f"])
            sq.soniq_mp_gemm_quantize_next(s["act_up"], s["up"], s["act_down"], s["s_next"])
            sq.soniq_mp_gemm(s["act_down"], s["down"], out=s["Y"])

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        step()
    torch.cuda.synchronize()
    return dict(kind=kind, blocks=blocks, graph=graph, out=[y for s in blocks for y in (s["Y_o"], s["Y"])])


# -------------------------------------------------------------------- pass

def run(state):
    kind = state["kind"]
    if kind == "linear":
        return sq.soniq_quantize_mp_gemm(state["act"], state["w"], state["A"], out=state["Y"])
    if kind == "conv":
        sq.soniq_quantize_act_conv3x3(state["act"], state["X"])
        return sq.soniq_mp_gemm(state["act"], state["w"], out=state["Y"])
    if kind == "ffn":
        sq.soniq_quantize_act(state["act_up"], state["A"])
        if state["static"]:
            sq.soniq_mp_gemm_quantize_next(state["act_up"], state["up"], state["act_down"], state["s_next"])
            return sq.soniq_mp_gemm(state["act_down"], state["down"], out=state["Y"])
        sq.soniq_mp_gemm_quantize_next_max(state["act_up"], state["up"], state["act_down"], out=state["H"])
        return state["H"], sq.soniq_mp_gemm(state["act_down"], state["down"], out=state["Y"])
    state["graph"].replay()
    return state["out"]


# ------------------------------------------------------------------ limits

def _linear_work(M, N, K, w, w_lo_share, reads_a=True, writes_y=True):
    n_lo = int(round(w_lo_share * N))
    w_bytes = K * (n_lo * w[0] + (N - n_lo) * w[1]) / 8 + 4 * N
    return dict(bytes=w_bytes + (4 * M * K if reads_a else 0) + (2 * M * N if writes_y else 0),
                flops=2.0 * M * N * K)


def work(case):
    """Inputs read once, weights at their own widths, outputs written once."""
    kind = case["kind"]
    if kind == "linear":
        parts = [_linear_work(case["M"], case["N"], case["K"], (case["w_lo"], case["w_hi"]), case["w_lo_share"])]
    elif kind == "conv":
        pixels, C, N = case["B"] * case["H"] * case["W"], case["C"], case["N"]
        p = _linear_work(pixels, N, 9 * C, (1, 4), 0.8, reads_a=False)
        p["bytes"] += 4 * pixels * C
        parts = [p]
    elif kind == "ffn":
        parts = [_linear_work(case["M"], case["F"], case["K"], (2, 8), 0.7, writes_y=not case["static"]),
                 _linear_work(case["M"], case["N"], case["F"], (2, 8), 0.7, reads_a=False)]
    else:
        M, K, F, w = case["M"], case["K"], case["F"], ((2, 4), 0.75)
        parts = [_linear_work(M, K, K, *w), _linear_work(M, F, K, *w, writes_y=False),
                 _linear_work(M, K, F, *w, reads_a=False)] * case["layers"]
    return {k: sum(p[k] for p in parts) for k in ("bytes", "flops")}


def tolerance(case):
    """The integer sums are exact, so two correct implementations differ where
    the fp32 scaling falls on the other side of a bf16 boundary (one step of
    2^-8 of the value) and where an fp32 quotient moves a code.  Measured
    against the same path in 64 bits, rounded to bf16: rel up to 2.1e-4, max
    0.05 for one layer; rel 5e-4, max 0.1 where a second layer takes its input
    from the first."""
    if case["kind"] in ("ffn", "stack"):
        return {"rel": 2e-3, "max": 0.4}
    return {"rel": 8e-4, "max": 0.2}


# ------------------------------------------------------------- 64-bit check

def _container(b):
    return 1 if b <= 1 else 2 if b <= 2 else 4 if b <= 4 else 8


def _codes(x, s, b, signed):
    """Codes of x (float64) with scale s: rint(x / s) within the width's range."""
    if b == 1 and signed:
        return torch.where(x >= 0, 1.0, -1.0).double()
    hi = float(2 ** (b - 1) - 1 if signed else 2 ** b - 1)
    return torch.nan_to_num(torch.round(x / s)).clamp_(-hi if signed else 0.0, hi)


def _top(b, signed):
    return 1.0 if b == 1 else float(2 ** (b - 1) - 1 if signed else 2 ** b - 1)


def _exact_weights(W, w_bits):
    out = torch.empty(W.shape, dtype=torch.float64, device="cuda")
    for b in sorted(set(w_bits.tolist())):
        rows = torch.from_numpy(np.flatnonzero(w_bits == b)).cuda()
        x = W[rows].double()
        s = x.abs().amax(1, keepdim=True) / _top(b, True)
        out[rows] = _codes(x, s, b, True) * s
    return out


def _exact_activations(A, a_bits, signed, group_bits=0, scales=None):
    """Quantized values, one scale per width (or per block of group_bits of
    one width's channels in their order), the largest value over the batch."""
    out = torch.empty(A.shape, dtype=torch.float64, device="cuda")
    for g, b in enumerate(sorted(set(a_bits.tolist()))):
        cols = np.flatnonzero(a_bits == b)
        n = group_bits // _container(b) if group_bits else len(cols)
        for i in range(0, len(cols), n):
            c = torch.from_numpy(cols[i:i + n]).cuda()
            x = A[:, c].double()
            s = x.abs().amax() / _top(b, signed) if scales is None else float(np.float32(scales[g]))
            out[:, c] = _codes(x, s, b, signed) * s
    return out


def _exact_linear(A, layer, signed=True, **more):
    return _exact_activations(A, layer["a_bits"], signed, **more) @ _exact_weights(layer["W"], layer["w_bits"]).T


def exact(case, seed):
    data = _data(case, seed)
    kind = case["kind"]
    if kind == "linear":
        return _exact_linear(data["A"], data["layer"], case["a_signed"], group_bits=case["group_bits"])
    if kind == "conv":
        X, F = data["X"], data["F"]
        B, C, H, W = X.shape
        q = _exact_activations(X.permute(0, 2, 3, 1).reshape(-1, C), data["c_bits"], False)
        q = torch.nn.functional.pad(q.reshape(B, H, W, C), (0, 0, 1, 1, 1, 1))
        f = _exact_weights(F.reshape(F.shape[0], -1), data["w_bits"]).reshape(F.shape)
        y = torch.zeros((B * H * W, F.shape[0]), dtype=torch.float64, device="cuda")
        for i in range(3):
            for j in range(3):
                y += q[:, i:i + H, j:j + W].reshape(-1, C) @ f[:, :, i, j].T.contiguous()
        return y
    if kind == "ffn":
        h = _exact_linear(data["A"], data["up"])
        if case["static"]:
            return _exact_linear(h, data["down"], scales=data["s_next"])
        # the second layer's input is defined on the stored bf16 values
        return h, _exact_linear(h.float().bfloat16(), data["down"])
    out = []
    for b in data["blocks"]:
        out.append(_exact_linear(b["x_o"], b["o"]))
        out.append(_exact_linear(_exact_linear(b["x_f"], b["up"]), b["down"], scales=b["s_next"]))
    return out
