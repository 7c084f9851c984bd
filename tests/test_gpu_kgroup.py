"""The K-group kernel (few to a few hundred bf16 rows) at the edges of its
shapes, against the fp64 oracle, and against the tiled exact kernel on the
same inputs.

Both add each block's partial (at most 32 products of exact operands) in
fp32, scaled by s, K / 32 times, and the K-group kernel adds up to 16 groups'
sums: element by element |Y - Y_ref| <= (K / 32 + 32 + 16) * 2^-24 *
(|X| |W_d|^T).
"""
import numpy as np
import pytest

import kgroup_cases as cases
import synth_inputs as si
from oracle import oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU (run with -m 'not gpu' on a CPU host)")
    from paper_2607_08526_amd import qlinear as ql
    ql.load()
    return torch, ql


def run(gpu, fmt, X, codes, scales, N, **ep):
    torch, ql = gpu
    dv = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    Y = ql.forward_ep(fmt, dv(X.view(np.int16)), dv(codes), dv(scales.view(np.int16)), N, **ep)
    torch.cuda.synchronize()
    return Y.float().cpu().numpy().astype(np.float64)


# rows around every staging size and row tile, columns around 32, 64 and 128
# and not a multiple of 4, one stage and a half-filled last stage, long K
@pytest.mark.parametrize("M,N,K", cases.SINGLES)
@pytest.mark.parametrize("fmt", [O.FMT_Q4, O.FMT_INT8])
def test_kgroup_shapes(gpu, orc, fmt, M, N, K):
    torch, ql = gpu
    W, X = si.small_case(8100 + M + N + K, M, N, K)
    codes, scales = orc.quantize(fmt, W)
    codes.reshape(-1)[:8] = [0x80, 0x88, 0x08, 0x7F, 0xFF, 0xF8, 0x8F, 0x00]  # -128 / -8 too
    Yr = orc.forward(fmt, X, O.DT_BF16, codes, scales, N)
    Wd = np.abs(orc.dequantize(fmt, codes, scales, N, K))
    B = (K // 32 + 48) * 2.0 ** -24 * (np.abs(si.bf16_bits_to_f32(X)).astype(np.float64) @ Wd.T)
    Yg = run(gpu, fmt, X, codes, scales, N)
    assert np.all(np.abs(Yg - Yr) <= B + 1e-30)
    with ql.forced_path(ql.PATH_TILED):
        Yt = run(gpu, fmt, X, codes, scales, N)
    assert np.all(np.abs(Yg - Yt) <= 2 * B + 1e-30)


@pytest.mark.parametrize("M,N,K", cases.SINGLES_F32_F16)
@pytest.mark.parametrize("kind", ["q4 f32", "int8 f32", "f16"])
def test_kgroup_fp32_and_fp16(gpu, orc, kind, M, N, K):
    """fp32 activations (three exact bf16 planes, six MFMAs per block) and fp16
    weights (X shifted to fp16, exact up to 2^-29 of the row's maximum), the
    same bound with 96 and 32 products per block."""
    torch, ql = gpu
    dv = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    f16 = kind == "f16"
    W, X = si.small_case(8400 + M + N + K, M, N, K, O.DT_BF16 if f16 else O.DT_F32)
    X[M - 1] = X[M - 1] if f16 else X[M - 1] * np.float32(1e-6)
    if f16:
        fmt, codes, scales, x = ql.FMT_F16, W.astype(np.float16), None, si.bf16_bits_to_f32(X)
        Wd, xd = codes.astype(np.float64), dv(X.view(np.int16))
    else:
        fmt = ql.FMT_Q4 if kind[:2] == "q4" else ql.FMT_INT8
        codes, scales = orc.quantize(fmt, W)
        Wd, x, xd = orc.dequantize(fmt, codes, scales, N, K), X, dv(X)
    Yr = x.astype(np.float64) @ Wd.T
    B = (K // 32 + 112) * 2.0 ** -24 * (np.abs(x).astype(np.float64) @ np.abs(Wd).T)
    Y = ql.forward(fmt, xd, dv(codes), None if f16 else dv(scales.view(np.int16)), N)
    torch.cuda.synchronize()
    assert np.all(np.abs(Y.cpu().numpy().astype(np.float64) - Yr) <= B + 1e-30)


@pytest.mark.parametrize("fmt,f32,M,layers,shapes", cases.GROUPS)
def test_kgroup_every_shape(gpu, orc, fmt, f32, M, layers, shapes):
    """Groups that cover every shape of every launch (kgroup_cases.py), every
    output NaN-filled, element by element within the bound above (fp32 X: 96
    products per block); a second call repeats the first bit for bit."""
    torch, ql = gpu
    dv = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    xdt = O.DT_F32 if f32 else O.DT_BF16
    ents, refs = [], []
    for i, (N, K) in enumerate(layers):
        W, X = si.small_case(8700 + i + M + N + K, M, N, K, xdt)
        x = X if f32 else si.bf16_bits_to_f32(X)
        if fmt == cases.F16:
            codes, scales = W.astype(np.float16), None
            Wd = codes.astype(np.float64)
        else:
            codes, scales = orc.quantize(fmt, W)
            Wd = orc.dequantize(fmt, codes, scales, N, K)
        Y = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
        ents.append((fmt, dv(X if f32 else X.view(np.int16)), dv(codes),
                     None if scales is None else dv(scales.view(np.int16)), N, Y))
        A = np.abs(x).astype(np.float64) @ np.abs(Wd).T
        refs.append((x.astype(np.float64) @ Wd.T, (K // 32 + 112) * 2.0 ** -24 * A + 1e-30))
    ql.block_forward(ents)
    torch.cuda.synchronize()
    first = [e[5].clone() for e in ents]
    ql.block_forward(ents)
    torch.cuda.synchronize()
    for e, Y1, (Yr, B), nk in zip(ents, first, refs, layers):
        assert torch.equal(e[5], Y1), nk
        assert np.all(np.abs(Y1.cpu().numpy().astype(np.float64) - Yr) <= B), nk


@pytest.mark.parametrize("M", [7, 30, 107])
def test_kgroup_block(gpu, orc, M):
    """A block of layers of different lengths and epilogues in one launch,
    every output NaN-filled; NaN and infinite activations stay in their rows."""
    torch, ql = gpu
    d = 512
    rng = np.random.default_rng(8300 + M)
    xs = {K: si.f32_to_bf16_bits(rng.standard_normal((M, K)).astype(np.float32)) for K in (d, 4 * d)}
    xs[d][1, 5], xs[d][2, 9] = 0x7FC0, 0x7F80
    dv = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    ents, refs = [], []
    for i, (_, N, K) in enumerate(si.block_linears(d)):
        codes, scales = orc.quantize(O.FMT_Q4, si.weights(rng, N, K))
        bias = rng.standard_normal(N).astype(np.float32)
        resid = rng.standard_normal((M, N)).astype(np.float32)
        act = O.ACT_GELU if i == 2 else O.ACT_NONE
        Y = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
        ents.append((ql.FMT_Q4, dv(xs[K].view(np.int16)), dv(codes), dv(scales.view(np.int16)), N,
                     Y, dv(bias), act, dv(resid)))
        keep = np.ones(M, bool)
        keep[1:3] = K != d
        P = orc.forward(O.FMT_Q4, xs[K][keep], O.DT_BF16, codes, scales, N)
        refs.append((keep, orc.epilogue(P, bias, act, resid[keep]), np.abs(P).max()))
    ql.block_forward_ep(ents)
    torch.cuda.synchronize()
    for e, (keep, ref, top) in zip(ents, refs):
        Y = e[5].cpu().numpy().astype(np.float64)
        assert np.all(np.abs(Y[keep] - ref) <= 1e-5 * top + 2e-6 * np.abs(ref) + 1e-6)
        assert not np.isfinite(Y[~keep]).any()


@pytest.mark.parametrize("fmt", [O.FMT_Q4, O.FMT_INT8])
def test_kgroup_fp32_large_activations(gpu, orc, fmt):
    """Activations so large that a block's sum of x * c, at most 32 of them,
    only just stays below the largest fp32 value: finite, and within the bound
    of test_kgroup_fp32_and_fp16.  (The tiled kernel takes them too.)"""
    torch, ql = gpu
    dv = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    M, N, K = 64, 1024, 1024
    W, X = si.small_case(8600 + fmt, M, N, K, O.DT_F32)
    codes, scales = orc.quantize(fmt, W)
    top = 3.4e38 / (32 * (7 if fmt == O.FMT_Q4 else 127))
    X = (X * (0.95 * top / np.abs(X).max())).astype(np.float32)
    Wd = orc.dequantize(fmt, codes, scales, N, K)
    Yr = X.astype(np.float64) @ Wd.T
    B = (K // 32 + 112) * 2.0 ** -24 * (np.abs(X).astype(np.float64) @ np.abs(Wd).T)
    outs = [ql.forward(fmt, dv(X), dv(codes), dv(scales.view(np.int16)), N)]
    with ql.forced_path(ql.PATH_TILED):
        outs.append(ql.forward(fmt, dv(X), dv(codes), dv(scales.view(np.int16)), N))
    torch.cuda.synchronize()
    for Y in outs:
        Y = Y.cpu().numpy().astype(np.float64)
        assert np.isfinite(Y).all()
        assert np.all(np.abs(Y - Yr) <= B)


@pytest.mark.parametrize("fmt", [O.FMT_Q4, O.FMT_INT8])
@pytest.mark.parametrize("M", [1, 4, 16, 48, 100, 300])
def test_activations_at_the_stated_limit(gpu, fmt, M):
    """bf16 activations of 7e34 with the largest codes, all of one sign: the
    size up to which every exact kernel's block sums fit fp32
    (include/qlinear.h), offset forms included.  Y is K x c s, from the library's
    own choice and from every exact kernel that takes the call, within the bound
    above, twice for the offset forms' larger codes (up to 255 for 127)."""
    torch, ql = gpu
    N, K, Q, s = 96, 512, 7 if fmt == O.FMT_Q4 else 127, 2.0 ** -10
    X = torch.full((M, K), 7e34, device="cuda").to(torch.bfloat16)
    scales = torch.full((N, K // 32), s, dtype=torch.float16, device="cuda").view(torch.int16)
    paths = [ql.PATH_AUTO, ql.PATH_TILED, ql.PATH_MID]
    paths += [ql.PATH_GEMV] if M <= 4 else []
    paths += [ql.PATH_STREAM, ql.PATH_SKINNY] if M <= 32 else []
    want = float(X[0, 0]) * K * Q * s
    for sign in (1, -1):
        if fmt == O.FMT_Q4:
            codes = torch.full((N, K // 2), 17 * (sign * Q & 15), dtype=torch.uint8, device="cuda")
        else:
            codes = torch.full((N, K), sign * Q, dtype=torch.int8, device="cuda").view(torch.uint8)
        for path in paths:
            with ql.forced_path(path):
                Y = ql.forward(fmt, X, codes, scales, N)
            torch.cuda.synchronize()
            err = np.abs(Y.cpu().numpy().astype(np.float64) - sign * want)
            assert np.all(err <= 2 * (K // 32 + 48) * 2.0 ** -24 * want), (path, sign)
