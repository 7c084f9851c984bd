"""Performance cases: the work a program has this library do, each through
the public entry points of `paper_2607_08526_amd.qlinear`.

    listed()            the cases themselves
    draw(rng)           one more case of the same ranges
    prepare(case, seed) inputs, weights, groups and graphs of one case
    run(state)          one pass; returns every output whole
    work(case)          bytes and flops a pass cannot do without
    tolerance(case)     how far another correct implementation may be
    exact(case, seed)   the outputs in 64-bit torch

Kinds of case:

  linear     one layer through forward_ep, called eagerly: one product of a
             program that does not group its layers
  step       a denoising step's linears: one grouped block_forward_ep call
             per DiT block, all blocks captured in one HIP graph, replayed
  dit        the chained denoising step (linears, attention, residual
             stream, steering) captured in one HIP graph, replayed
  attention  the fused attention on a fused QKV tensor, called eagerly
  w8a8       one block in the 8-bit-arithmetic mode: per-token quantization
             of every layer's input and the four int8 products, eagerly
  quantize   compression of one weight (load time)

Weights are N(0, 0.02) and activations N(0, 1), as in synth_inputs.py, drawn
on the GPU; the chained step scales its residual-branch weights by
1 / sqrt(2 blocks), as transformers are initialised, so that the residual
stream keeps the size it has in a trained model.
"""
import math

import torch

from paper_2607_08526_amd import qlinear as ql

FMT = {"q4": ql.FMT_Q4, "int8": ql.FMT_INT8, "f16": ql.FMT_F16}
QMAX = {"q4": 7, "int8": 127}
STEER = (12.0, 0.15)  # mean residual norm and strength of the chained step


def listed():
    return [
        # the smallest: one int8 layer on fp32 activations (a conditioning
        # projection), 64 rows of width 1024
        {"name": "linear int8 fp32", "kind": "linear", "fmt": "int8", "x": "f32", "M": 64,
         "N": 1024, "K": 1024, "ep": "none"},
        # the 4-bit FFN-up layer of the d = 1536 model with its epilogue, at
        # 256 tokens
        {"name": "linear q4 mid", "kind": "linear", "fmt": "q4", "x": "bf16", "M": 256,
         "N": 6144, "K": 1536, "ep": "gelu"},
        # unquantized fp16 weights (the reference precision) at the 214
        # tokens of a 10 s clip, the QKV layer of the d = 1536 model
        {"name": "linear f16 clip", "kind": "linear", "fmt": "f16", "x": "bf16", "M": 214,
         "N": 4608, "K": 1536, "ep": "bias"},
        # few rows: latency and weight bandwidth.  One row
        {"name": "step int8 1 row", "kind": "step", "fmt": "int8", "M": 1, "d": 2048,
         "blocks": 24, "ep": "none"},
        # a handful of rows, the 4-bit weights
        {"name": "step q4 8 rows", "kind": "step", "fmt": "q4", "M": 8, "d": 2048,
         "blocks": 24, "ep": "none"},
        # a few dozen rows, a ragged count, the d = 1536 model
        {"name": "step q4 27 rows", "kind": "step", "fmt": "q4", "M": 27, "d": 1536,
         "blocks": 24, "ep": "full"},
        # the d = 1024 model's whole denoising step on a 10 s clip (two
        # guidance branches of 107 latent frames)
        {"name": "dit q4 clip", "kind": "dit", "fmt": "q4", "B": 2, "T": 107, "d": 1024,
         "blocks": 20},
        # large batches: 8-bit blocks at 2048 tokens, linears only
        {"name": "step int8 2048 rows", "kind": "step", "fmt": "int8", "M": 2048, "d": 2048,
         "blocks": 8, "ep": "none"},
        # the largest: the d = 2048 model's whole denoising step, 4-bit
        # weights, two guidance branches of 1024 latent frames
        {"name": "dit q4 long", "kind": "dit", "fmt": "q4", "B": 2, "T": 1024, "d": 2048,
         "blocks": 24},
        # attention of a 60 s clip (645 latent frames, ragged) at d = 1536
        {"name": "attention 60 s", "kind": "attention", "B": 2, "T": 645, "H": 24, "o": "bf16"},
        # the 60 s clip in the 8-bit-arithmetic mode, one block at d = 1536
        {"name": "w8a8 60 s", "kind": "w8a8", "M": 1290, "d": 1536, "ep": "full"},
        # load time: one FFN-up weight to 4 bits
        {"name": "quantize q4", "kind": "quantize", "fmt": "q4", "N": 8192, "K": 2048},
    ]


def _log(rng, lo, hi):
    """An integer in [lo, hi], uniform in its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["linear", "linear", "step", "step", "dit", "attention", "w8a8",
                       "quantize"])
    if kind == "linear":
        fmt = rng.choice(["q4", "int8", "q4", "int8", "f16"])
        x = "bf16" if fmt == "f16" else rng.choice(["bf16", "bf16", "f32"])
        # whole 256-column widths as in the models, or any multiple of a block
        K = 256 * _log(rng, 1, 32) if fmt == "f16" or rng.random() < 0.7 \
            else 32 * _log(rng, 8, 256)
        return {"kind": kind, "fmt": fmt, "x": x, "M": _log(rng, 1, 2100),
                "N": _log(rng, 64, 8200), "K": K,
                "ep": rng.choice(["none", "bias", "gelu", "full"])}
    if kind == "step":
        return {"kind": kind, "fmt": rng.choice(["q4", "int8"]), "M": _log(rng, 1, 2048),
                "d": rng.choice([512, 768, 1024, 1152, 1536, 2048]),
                "blocks": rng.randint(4, 24), "ep": rng.choice(["none", "full"])}
    if kind == "dit":
        return {"kind": kind, "fmt": rng.choice(["q4", "int8"]), "B": rng.randint(1, 2),
                "T": _log(rng, 12, 1024), "d": rng.choice([512, 768, 1024, 1536, 2048]),
                "blocks": rng.randint(4, 24)}
    if kind == "attention":
        return {"kind": kind, "B": rng.randint(1, 4), "T": _log(rng, 40, 4096),
                "H": rng.randint(8, 32), "o": rng.choice(["bf16", "f32"])}
    if kind == "w8a8":
        return {"kind": kind, "M": _log(rng, 32, 2100),
                "d": rng.choice([512, 768, 1024, 1152, 1536, 2048]),
                "ep": rng.choice(["none", "full"])}
    return {"kind": kind, "fmt": rng.choice(["q4", "int8"]), "N": _log(rng, 512, 8200),
            "K": 32 * _log(rng, 16, 256)}


# ---- inputs (shared by prepare and exact: the same seed, the same values) ----

class _Draw:
    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)

    def normal(self, *shape, std=1.0):
        return torch.randn(shape, generator=self.g, device="cuda") * std

    def weight(self, fmt, N, K, std=0.02):
        W = self.normal(N, K, std=std)
        return W.to(torch.float16) if fmt == "f16" else W


def _layers(d):
    """(N, K) of a block's QKV, attention output, FFN-up and FFN-down."""
    return [(3 * d, d), (d, d), (4 * d, d), (d, 4 * d)]


def _has(ep):
    """(bias, GELU, residual) of an epilogue's name."""
    return ep != "none", ep in ("gelu",), ep == "full"


def _linear_inputs(case, seed):
    r = _Draw(seed)
    M, N, K = case["M"], case["N"], case["K"]
    W = r.weight(case["fmt"], N, K)
    X = r.normal(M, K)
    X = X if case["x"] == "f32" else X.to(torch.bfloat16)
    bias, _, resid = _has(case["ep"])
    return W, X, r.normal(N, std=0.1) if bias else None, r.normal(M, N) if resid else None


def _step_inputs(case, seed):
    """Two activation tensors shared by every block, then block by block its
    four weights and, with an epilogue, their biases; the residual of the
    out-projection and FFN-down."""
    r = _Draw(seed)
    M, d = case["M"], case["d"]
    xa, xb = r.normal(M, d).to(torch.bfloat16), r.normal(M, 4 * d).to(torch.bfloat16)
    h = r.normal(M, d) if case["ep"] == "full" else None

    def blocks():
        for _ in range(case["blocks"]):
            yield [(r.weight(case["fmt"], N, K),
                    r.normal(N, std=0.1) if case["ep"] == "full" else None)
                   for N, K in _layers(d)]

    return xa, xb, h, blocks()


def _dit_inputs(case, seed):
    r = _Draw(seed)
    M, d, n = case["B"] * case["T"], case["d"], case["blocks"]
    h0 = r.normal(M, d)
    direction = r.normal(d)
    direction /= direction.norm()
    stds = [0.02, 0.02 / math.sqrt(2 * n), 0.02, 0.02 / math.sqrt(2 * n)]

    def blocks():
        for _ in range(n):
            yield [(r.weight(case["fmt"], N, K, std), r.normal(N, std=0.1))
                   for (N, K), std in zip(_layers(d), stds)]

    return h0, direction, blocks()


def _attention_inputs(case, seed):
    return _Draw(seed).normal(case["B"] * case["T"], 3 * 64 * case["H"]).to(torch.bfloat16)


def _w8a8_inputs(case, seed):
    r = _Draw(seed)
    M, d, full = case["M"], case["d"], case["ep"] == "full"
    layers = []
    for i, (N, K) in enumerate(_layers(d)):
        layers.append((r.normal(N, K, std=0.02), r.normal(M, K).to(torch.bfloat16),
                       r.normal(N, std=0.1) if full else None,
                       r.normal(M, N) if full and i in (1, 3) else None))
    return layers


# ---- prepare and run -------------------------------------------------------

def _compress(fmt, W):
    """(codes, scales) a program keeps of a weight."""
    return (W, None) if fmt == "f16" else ql.quantize(FMT[fmt], W)


_STREAM = []


def _capture(fn):
    """fn's launches as a HIP graph.  One stream for every capture: it runs
    fn once first, so the library's workspace of that stream has its size."""
    if not _STREAM:
        _STREAM.append(torch.cuda.Stream())
    s = _STREAM[0]
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        fn()
    torch.cuda.current_stream().wait_stream(s)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        fn()
    return g


def _prepare_linear(case, seed):
    W, X, bias, resid = _linear_inputs(case, seed)
    codes, scales = _compress(case["fmt"], W)
    act = ql.ACT_GELU if _has(case["ep"])[1] else ql.ACT_NONE
    return {"args": (FMT[case["fmt"]], X, codes, scales, case["N"]),
            "kw": dict(bias=bias, act=act, residual=resid,
                       ydtype=torch.bfloat16 if case["ep"] == "gelu" else torch.float32)}


def _prepare_step(case, seed):
    xa, xb, h, blocks = _step_inputs(case, seed)
    M, full, n = case["M"], case["ep"] == "full", case["blocks"]
    # QKV and FFN-up leave as bf16 with an epilogue: attention and FFN-down
    # read them
    dts = [torch.bfloat16 if full and i in (0, 2) else torch.float32 for i in range(4)]
    Y = [torch.empty((n, M, N), dtype=dt, device="cuda")
         for (N, _), dt in zip(_layers(case["d"]), dts)]
    groups = []
    for b, layers in enumerate(blocks):
        ents = []
        for i, (W, bias) in enumerate(layers):
            codes, scales = _compress(case["fmt"], W)
            ents.append((FMT[case["fmt"]], xb if i == 3 else xa, codes, scales, W.shape[0],
                         Y[i][b], bias, ql.ACT_GELU if full and i == 2 else ql.ACT_NONE,
                         h if full and i in (1, 3) else None))
        groups.append(ql.make_group_ep(ents))

    def fn():
        for g in groups:
            ql.block_forward_ep(None, group=g)

    return {"graph": _capture(fn), "groups": groups, "out": Y}


def _prepare_dit(case, seed):
    h0, direction, blocks = _dit_inputs(case, seed)
    fmt, B, T, d = FMT[case["fmt"]], case["B"], case["T"], case["d"]
    M, H = B * T, d // 64
    empty = lambda n, dt: torch.empty((M, n), dtype=dt, device="cuda")
    qkv, att, up = (empty(n, torch.bfloat16) for n in (3 * d, d, 4 * d))
    h, hb = empty(d, torch.float32), empty(d, torch.bfloat16)
    hb0 = h0.to(torch.bfloat16)
    strength = torch.full((1,), STEER[1], device="cuda")
    calls = []
    for b, layers in enumerate(blocks):
        (c0, s0, b0), (c1, s1, b1), (c2, s2, b2), (c3, s3, b3) = \
            [(*_compress(case["fmt"], W), bias) for W, bias in layers]
        x_in, h_in = (hb0, h0) if b == 0 else (hb, h)
        steer = (direction, STEER[0], strength) if b == case["blocks"] // 2 else None
        calls.append([ql.make_group_ep([e]) for e in (
            (fmt, x_in, c0, s0, 3 * d, qkv, b0, ql.ACT_NONE, None),
            (fmt, att, c1, s1, d, h, b1, ql.ACT_NONE, h_in, None, hb),
            (fmt, hb, c2, s2, 4 * d, up, b2, ql.ACT_GELU, None),
            (fmt, up, c3, s3, d, h, b3, ql.ACT_NONE, h, steer, hb))])
    q, k, v = qkv[:, :d], qkv[:, d:2 * d], qkv[:, 2 * d:]

    def fn():
        for g0, g1, g2, g3 in calls:
            ql.block_forward_ep(None, group=g0)
            ql.attention(q, k, v, B, T, H, O=att)
            for g in (g1, g2, g3):
                ql.block_forward_ep(None, group=g)

    return {"graph": _capture(fn), "groups": calls, "qkv": qkv,
            "out": {"h": h, "hb": hb, "att": att, "up": up}}


def _prepare_attention(case, seed):
    qkv = _attention_inputs(case, seed)
    n = 64 * case["H"]
    return {"args": (qkv[:, :n], qkv[:, n:2 * n], qkv[:, 2 * n:], case["B"], case["T"], case["H"]),
            "O": torch.empty((qkv.shape[0], n), device="cuda",
                             dtype=torch.bfloat16 if case["o"] == "bf16" else torch.float32)}


def _prepare_w8a8(case, seed):
    full, M = case["ep"] == "full", case["M"]
    layers = []
    for i, (W, X, bias, resid) in enumerate(_w8a8_inputs(case, seed)):
        N, K = W.shape
        codes, scales = ql.quantize(ql.FMT_INT8, W)
        layers.append({
            "X": X, "qx": torch.empty((M, K), dtype=torch.int8, device="cuda"),
            "sx": torch.empty(M, dtype=torch.int16, device="cuda"),
            "codes": codes, "scales": scales, "N": N,
            "kw": dict(Y=torch.empty((M, N), device="cuda", dtype=torch.bfloat16
                                     if full and i in (0, 2) else torch.float32),
                       bias=bias, act=ql.ACT_GELU if full and i == 2 else ql.ACT_NONE,
                       residual=resid)})
    return {"layers": layers}


def _prepare_quantize(case, seed):
    W = _Draw(seed).normal(case["N"], case["K"], std=0.02)
    fmt = FMT[case["fmt"]]
    return {"fmt": fmt, "W": W, "codes": ql.empty_codes(fmt, case["N"], case["K"]),
            "scales": ql.empty_scales(case["N"], case["K"])}


def prepare(case, seed):
    state = {"linear": _prepare_linear, "step": _prepare_step, "dit": _prepare_dit,
             "attention": _prepare_attention, "w8a8": _prepare_w8a8,
             "quantize": _prepare_quantize}[case["kind"]](case, seed)
    state["kind"] = case["kind"]
    return state


def run(state):
    kind = state["kind"]
    if kind in ("step", "dit"):
        state["graph"].replay()
        return state["out"]
    if kind == "linear":
        return ql.forward_ep(*state["args"], **state["kw"])
    if kind == "attention":
        return ql.attention(*state["args"], O=state["O"])
    if kind == "quantize":
        codes, scales = ql.quantize(state["fmt"], state["W"], state["codes"], state["scales"])
        return {"codes": codes, "scales": scales}
    out = []
    for l in state["layers"]:
        qx, sx = ql.quantize_act(l["X"], l["qx"], l["sx"])
        out.append({"qx": qx, "sx": sx,
                    "Y": ql.forward_w8a8(qx, sx, l["codes"], l["scales"], l["N"], **l["kw"])})
    return out


# ---- work and tolerance ----------------------------------------------------

def _weight_bytes(fmt, N, K):
    return 2 * N * K if fmt == "f16" else N * K // (2 if fmt == "q4" else 1) + N * K // 16


def work(case):
    kind = case["kind"]
    if kind == "linear":
        M, N, K = case["M"], case["N"], case["K"]
        bias, gelu, resid = _has(case["ep"])
        b = _weight_bytes(case["fmt"], N, K) + M * K * (4 if case["x"] == "f32" else 2)
        b += M * N * ((2 if gelu else 4) + (4 if resid else 0)) + (4 * N if bias else 0)
        return {"bytes": b, "flops": 2 * M * N * K}
    if kind in ("step", "dit"):
        d, n = case["d"], case["blocks"]
        M = case["M"] if kind == "step" else case["B"] * case["T"]
        params = 12 * d * d
        b = n * sum(_weight_bytes(case["fmt"], N, K) for N, K in _layers(d))
        flops = n * 2 * M * params
        if kind == "step" and case["ep"] == "none":
            b += M * 5 * d * 2 + n * M * 9 * d * 4
        elif kind == "step":
            b += M * 5 * d * 2 + M * d * 4 + n * (9 * d * 4 + M * (7 * d * 2 + 2 * d * 4))
        else:
            # within a pass the activations may stay on the chip: the input,
            # the biases and the four returned buffers are what remains
            b += M * d * 4 + n * 9 * d * 4 + M * (d * 6 + d * 2 + 4 * d * 2)
            flops += n * 4 * M * case["T"] * d
        return {"bytes": b, "flops": flops}
    if kind == "attention":
        M, n = case["B"] * case["T"], 64 * case["H"]
        return {"bytes": M * n * (6 + (2 if case["o"] == "bf16" else 4)),
                "flops": 4 * M * case["T"] * n}
    if kind == "w8a8":
        M, d, full = case["M"], case["d"], case["ep"] == "full"
        b = 12 * d * d + 12 * d * d // 16 + M * 7 * d * 3 + 8 * M
        b += M * (7 * d * 2 + 2 * d * 8) + 36 * d if full else M * 9 * d * 4
        return {"bytes": b, "flops": 2 * M * 12 * d * d}
    N, K = case["N"], case["K"]
    return {"bytes": 4 * N * K + _weight_bytes(case["fmt"], N, K), "flops": N * K}


def tolerance(case):
    """About four times the error against exact() that the kernels show."""
    kind = case["kind"]
    if kind == "quantize":
        return "exact"
    if kind == "dit":  # 0.003, bf16 roundings through all the blocks
        return {"rel": 1.2e-2, "max": 0.3}
    if kind == "attention":  # 0.0023: bf16 probabilities
        return {"rel": 1e-2, "max": 0.1}
    bf16_out = {"rel": 7e-3, "max": 0.05, "differ": 0.0}  # 0.0017: one bf16 rounding
    fp32_sum = {"rel": 2e-6, "max": 2e-5, "differ": 0.0}  # 1e-7 to 5e-7
    if kind == "w8a8":
        return bf16_out if case["ep"] == "full" else fp32_sum
    if case["ep"] == ("gelu" if kind == "linear" else "full"):
        return bf16_out
    if kind == "linear" and (case["x"] == "f32" or case["K"] % 256):
        return fp32_sum
    # above 64 rows a weight may be rounded once to fp16: 2e-4
    return {"rel": 1e-3, "max": 1e-2} if case["M"] > 64 else fp32_sum


# ---- the same in 64 bits ---------------------------------------------------

def _dequant(fmt, W):
    """The fp64 weight that `fmt` stores of the fp32 W (for f16: W itself)."""
    W = W.double()
    if fmt == "f16":
        return W
    codes, scales = _codes(fmt, W)
    return (codes.view(W.shape[0], -1, 32) * scales[:, :, None]).view(W.shape)


def _codes(fmt, W):
    """(codes [N][K], scales [N][K/32]) of fp64 W by the format's rule, fp64."""
    blocks = W.view(W.shape[0], -1, 32)
    scales = (blocks.abs().amax(-1) / QMAX[fmt]).half().double()
    codes = torch.where(scales[:, :, None] > 0, blocks / scales[:, :, None], 0.0)
    return codes.round().clamp(-QMAX[fmt], QMAX[fmt]).view(W.shape), scales


def _finish(Y, bias=None, gelu=False, resid=None):
    if bias is not None:
        Y = Y + bias.double()
    if gelu:
        Y = torch.nn.functional.gelu(Y)
    return Y if resid is None else Y + resid.double()


def _attention64(qkv, B, T, H):
    q, k, v = (t.view(B, T, H, 64).transpose(1, 2).contiguous()
               for t in qkv.split(64 * H, dim=1))
    out = []
    for b in range(B):  # one sequence at a time: the scores are T x T per head
        p = torch.softmax(torch.matmul(q[b], k[b].transpose(1, 2).contiguous()) / 8.0, -1)
        out.append(torch.matmul(p, v[b]))
    return torch.stack(out).transpose(1, 2).reshape(B * T, 64 * H)


def exact(case, seed):
    kind = case["kind"]
    if kind == "linear":
        W, X, bias, resid = _linear_inputs(case, seed)
        return _finish(X.double() @ _dequant(case["fmt"], W).T, bias, _has(case["ep"])[1], resid)
    if kind == "step":
        xa, xb, h, blocks = _step_inputs(case, seed)
        xa, xb, full = xa.double(), xb.double(), case["ep"] == "full"
        out = [[], [], [], []]
        for layers in blocks:
            for i, (W, bias) in enumerate(layers):
                P = (xb if i == 3 else xa) @ _dequant(case["fmt"], W).T
                out[i].append(_finish(P, bias, full and i == 2,
                                      h if full and i in (1, 3) else None))
        return [torch.stack(o) for o in out]
    if kind == "dit":
        h, direction, blocks = _dit_inputs(case, seed)
        h = h.double()
        for b, layers in enumerate(blocks):
            (W0, b0), (W1, b1), (W2, b2), (W3, b3) = \
                [(_dequant(case["fmt"], W), bias) for W, bias in layers]
            att = _attention64(_finish(h @ W0.T, b0), case["B"], case["T"], case["d"] // 64)
            h = _finish(att @ W1.T, b1, resid=h)
            up = _finish(h @ W2.T, b2, gelu=True)
            h = _finish(up @ W3.T, b3, resid=h)
            if b == case["blocks"] // 2:
                h = h + STEER[1] * STEER[0] * direction.double()
        return {"h": h, "hb": h, "att": att, "up": up}
    if kind == "attention":
        return _attention64(_attention_inputs(case, seed).double(), case["B"], case["T"],
                            case["H"])
    if kind == "w8a8":
        out = []
        for i, (W, X, bias, resid) in enumerate(_w8a8_inputs(case, seed)):
            X = X.double()
            sx = (X.abs().amax(1, keepdim=True) / 127).half().double()
            qx = (X / sx).round().clamp(-127, 127)
            Y = (sx * qx) @ _dequant("int8", W).T
            out.append({"qx": None, "sx": None,
                        "Y": _finish(Y, bias, case["ep"] == "full" and i == 2, resid)})
        return out
    return None  # whole numbers only
