// Block quantizer: fp32 weights -> int8 or 4-bit codes + fp16 scales.
//
// Paper (Methodology, "Quantization and its evaluation"): the transformer's
// weights are compressed to 8-bit or 4-bit integers; the compressed copy then
// replaces the full-precision one.  Encoding used here: symmetric absmax over
// blocks of 32 weights along K, scale = fp16 nearest to absmax / Q (one
// rounding of the exact quotient, ties to even), code = nearest integer to
// w / scale (ties to even) clamped to [-Q, Q]; Q = 127 (int8) or 7 (q4).
//
// Exactness: neither quotient is formed.  An fp32 estimate of the scale is
// corrected by comparing absmax with exact midpoints (scale_bits), one of a
// code by its exact remainder (nearest_code).
//
// Bound: HBM (4.6 to 5.1 bytes per weight).  With an fp64 division per weight
// the VALU bound it instead: 8192 x 2048 to q4 23.5 us, 14.3 us now (5.3 TB/s).
//
// Layout: 4 lanes per 32-weight block, 8 consecutive weights per lane (two
// 16-byte loads); the 4 lanes of a block are adjacent in a wavefront and
// combine their absmax with two butterfly shuffles.
#include "internal.h"

namespace qlk {
namespace {

// Exact value of an fp16 bit pattern with the sign bit clear; 0x7C00 as 2^16,
// where the next normal would be.
__device__ inline float f16_value(uint32_t h)
{
    return h >= 0x7C00u ? 65536.0f : (float)__builtin_bit_cast(_Float16, (uint16_t)h);
}

// fp16 bit pattern nearest to amax / Q for a finite fp32 amax >= 0 (ties to
// even, subnormals kept, 0x7C00 when it rounds past 65504), exact: the fp32
// product with 1 / Q rounds to the right pattern or to a neighbour, and the
// midpoints to both neighbours times Q (12 and 7 significant bits) are exact
// in fp32, to be compared with amax itself.
template <int Q>
__device__ inline uint32_t scale_bits(float amax)
{
    const uint32_t h =
        __builtin_bit_cast(uint16_t, (_Float16)(amax * (1.0f / (float)Q)));  // overflow: 0x7C00
    const float v = f16_value(h);
    const float hi = (v + f16_value(h + 1)) * (0.5f * Q);
    const float lo = (v + f16_value(h - 1)) * (0.5f * Q);
    const bool odd = h & 1;
    if (h < 0x7C00u && (amax > hi || (amax == hi && odd)))
        return h + 1;
    if (h > 0 && (amax < lo || (amax == lo && odd)))
        return h - 1;
    return h;
}

// The integer nearest to w / s, ties to even, clamped to [-Q, Q], for s > 0 an
// fp16 value, |w| < 2^8 s and inv within 2 ulp of 1 / s; exact.  (|w| is at
// most Q (1 + 2^-11) s for a normal scale, and 1.5 Q s for a subnormal one,
// which may round down by a third; the clamp takes the excess.)
//   n = rint(w * inv) is within one of it: the product is off by less than
// 2^-21 of itself, 2^-13.  The remainder r = w - n s, at most s / 2 + 2^-13 s in
// size wherever it decides, is then compared with s / 2: above, n moves towards
// w; at the tie, n moves if it is odd.  r is exact in fp32.  With 2^E <= s <
// 2^(E+1): for n = 0 it is w; otherwise |w| > s / 2 (1 - 2^-21), so w and n s
// are multiples of 2^(E-24) and r, below 2^E, has 24 bits, unless s = 2^E and
// |w| is just below s / 2: there n = +-1 and r rounds to s / 2 or more, and n
// moves to 0 either way, as it has to.
__device__ inline int nearest_code(float w, float s, float inv, float half_s, int Q)
{
    const float n = __builtin_rintf(w * inv);
    const float r = __builtin_fmaf(-n, s, w);
    const float a = __builtin_fabsf(r);
    int c = (int)n;
    if (a > half_s || (a == half_s && (c & 1)))
        c += r > 0.0f ? 1 : -1;
    c = c > Q ? Q : c;
    return c < -Q ? -Q : c;
}

// The same for a bf16 x and Q = 127.  x has 8 significant bits and s 11, so that
// a quotient above 1/4 that is no half-integer is at least 2^-12 from every one
// (170 / 1.9208984375 = 88.50025...), while an fp32 quotient below 2^8 within an
// ulp is within 2^-16 of it; exact half-integers are representable.  One Newton
// step on x * inv with its exact remainder gives the quotient at every
// half-integer, and within an ulp elsewhere.
__device__ inline int nearest_code_bf16(float x, float s, float inv)
{
    const float q = x * inv;
    const float r = __builtin_fmaf(__builtin_fmaf(-q, s, x), inv, q);
    return (int)__builtin_amdgcn_fmed3f(__builtin_rintf(r), -127.0f, 127.0f);
}

// 1 / s for an fp16 s > 0 (2^-24 to 65504, so neither overflows nor underflows)
__device__ inline float inverse(float s) { return __builtin_amdgcn_rcpf(s); }

template <int FMT>
__global__ __launch_bounds__(256) void quantize_kernel(const float *__restrict__ W,
                                                       int64_t n_blocks,
                                                       uint8_t *__restrict__ codes,
                                                       uint16_t *__restrict__ scales,
                                                       int *__restrict__ status)
{
    constexpr int Q = FMT == QL_FMT_INT8 ? 127 : 7;
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t blk = t >> 2;  // row-major block index n * (K/32) + b
    const int part = (int)(t & 3);
    const bool valid = blk < n_blocks;

    uint32_t wb[8];
    if (valid) {
        const uint4 *p = reinterpret_cast<const uint4 *>(W + blk * 32 + part * 8);
        const uint4 a = p[0], b = p[1];
        wb[0] = a.x; wb[1] = a.y; wb[2] = a.z; wb[3] = a.w;
        wb[4] = b.x; wb[5] = b.y; wb[6] = b.z; wb[7] = b.w;
    } else {
#pragma unroll
        for (int j = 0; j < 8; ++j)
            wb[j] = 0;
    }

    // |w| compared as unsigned integers (monotone for non-NaN fp32 bit
    // patterns); anything at or above the +inf pattern is a NaN or Inf.
    uint32_t amax = 0;
    bool bad = false;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const uint32_t a = wb[j] & 0x7FFFFFFFu;
        bad |= a >= 0x7F800000u;
        amax = a > amax ? a : amax;
    }
    {
        const uint32_t o1 = (uint32_t)__shfl_xor((int)amax, 1);
        amax = o1 > amax ? o1 : amax;
        const uint32_t o2 = (uint32_t)__shfl_xor((int)amax, 2);
        amax = o2 > amax ? o2 : amax;
    }
    if (!valid)
        return;
    if (amax >= 0x7F800000u) {  // some lane of this block saw a NaN/Inf
        if (bad)
            *status = QL_ERR_RANGE;
        return;
    }

    const uint32_t sbits = scale_bits<Q>(__uint_as_float(amax));
    if (sbits == 0x7C00) {
        if (part == 0)
            *status = QL_ERR_RANGE;
        return;
    }
    const float s = f16_value(sbits);
    const float inv = inverse(s), half_s = 0.5f * s;

    int c[8];
#pragma unroll
    for (int j = 0; j < 8; ++j)
        c[j] = sbits == 0 ? 0 : nearest_code(__uint_as_float(wb[j]), s, inv, half_s, Q);

    if (part == 0)
        scales[blk] = (uint16_t)sbits;
    if (FMT == QL_FMT_INT8) {
        uint32_t lo = 0, hi = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            lo |= (uint32_t)(c[j] & 0xFF) << (8 * j);
            hi |= (uint32_t)(c[j + 4] & 0xFF) << (8 * j);
        }
        *reinterpret_cast<uint2 *>(codes + blk * 32 + part * 8) = make_uint2(lo, hi);
    } else {
        uint32_t word = 0;
#pragma unroll
        for (int j = 0; j < 8; ++j)
            word |= (uint32_t)(c[j] & 0xF) << (4 * j);
        *reinterpret_cast<uint32_t *>(codes + blk * 16 + part * 4) = word;
    }
}

// Per-token activation quantizer of the W8A8 path.  Scale = fp16 nearest to
// (row absmax) / 127 and code = nearest integer to x / scale clamped to
// [-127, 127] (the weight rules with the whole row as the block).  A row
// holding a NaN or Inf, or whose scale would overflow fp16, gets the NaN scale
// 0x7E00 and zero codes, so its outputs come out NaN.
//
// Bound: HBM at many rows, the load latency at few.  A workgroup per row
// keeps up to R groups of 8 columns per thread in registers between the
// maximum and the codes, so rows up to 8192 columns are read once.  (A
// wavefront per row was slower: 1290 x 1536 6.6 us.)  bf16, against two reads,
// an fp64 scale and a division per element: 1290 x 1536 4.5 -> 3.9 us, 1290 x
// 6144 9.4 -> 7.0 us (3.4 TB/s), 2048 x 8192 15.8 -> 12.3 us (4.1 TB/s).
template <bool BF16>
__device__ inline void load8(const void *X, int64_t e, uint32_t (&v)[8])
{
    if constexpr (BF16) {
        const uint4 a = *reinterpret_cast<const uint4 *>(static_cast<const uint16_t *>(X) + e);
        const uint32_t w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            v[2 * j] = w[j] << 16;
            v[2 * j + 1] = w[j] & 0xFFFF0000u;
        }
    } else {
        const uint4 *p = reinterpret_cast<const uint4 *>(static_cast<const float *>(X) + e);
        const uint4 a = p[0], b = p[1];
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
        v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    }
}

template <bool BF16, int R>
__global__ __launch_bounds__(256) void act_quant_kernel(const void *__restrict__ X, int64_t K,
                                                        int8_t *__restrict__ q,
                                                        uint16_t *__restrict__ sx)
{
    constexpr int T = 256;
    __shared__ uint32_t wmax[T / 64];
    const int64_t m = blockIdx.x, row = m * K;
    const int t = threadIdx.x;
    const int64_t groups = K / 8;
    uint32_t v[R][8];
    uint32_t amax = 0;  // |x| bit patterns compare like the values; NaN/Inf >= 0x7F800000
    auto max8 = [&](const uint32_t(&x)[8]) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t a = x[j] & 0x7FFFFFFFu;
            amax = a > amax ? a : amax;
        }
    };
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const int64_t g = t + (int64_t)i * T;
        if (g < groups) {
            load8<BF16>(X, row + 8 * g, v[i]);
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j)
                v[i][j] = 0;
        }
    }
#pragma unroll
    for (int i = 0; i < R; ++i)
        max8(v[i]);
    for (int64_t g = t + (int64_t)R * T; g < groups; g += T) {
        uint32_t x[8];
        load8<BF16>(X, row + 8 * g, x);
        max8(x);
    }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t w = (uint32_t)__shfl_xor((int)amax, o);
        amax = w > amax ? w : amax;
    }
    if ((t & 63) == 0)
        wmax[t >> 6] = amax;
    __syncthreads();
    amax = wmax[0];
#pragma unroll
    for (int w = 1; w < T / 64; ++w)
        amax = wmax[w] > amax ? wmax[w] : amax;

    uint32_t sbits = 0x7C00;
    if (amax < 0x7F800000u)
        sbits = scale_bits<127>(__uint_as_float(amax));
    const bool zero = sbits == 0x7C00 || sbits == 0;
    if (t == 0)
        sx[m] = (uint16_t)(sbits == 0x7C00 ? 0x7E00 : sbits);
    const float s = zero ? 1.0f : f16_value(sbits);
    const float inv = inverse(s), half_s = 0.5f * s;
    auto put8 = [&](int64_t g, const uint32_t(&x)[8]) {
        uint32_t c[8];
#pragma unroll
        for (int j = 0; j < 8; ++j)
            c[j] = zero ? 0u
                        : (uint32_t)(BF16 ? nearest_code_bf16(__uint_as_float(x[j]), s, inv)
                                          : nearest_code(__uint_as_float(x[j]), s, inv, half_s,
                                                         127)) & 0xFFu;
        *reinterpret_cast<uint2 *>(q + row + 8 * g) =
            make_uint2(c[0] | c[1] << 8 | c[2] << 16 | c[3] << 24,
                       c[4] | c[5] << 8 | c[6] << 16 | c[7] << 24);
    };
#pragma unroll
    for (int i = 0; i < R; ++i)
        if (t + (int64_t)i * T < groups)
            put8(t + (int64_t)i * T, v[i]);
    for (int64_t g = t + (int64_t)R * T; g < groups; g += T) {
        uint32_t x[8];
        load8<BF16>(X, row + 8 * g, x);
        put8(g, x);
    }
}

template <bool BF16>
void act_quant(const void *X, int64_t M, int64_t K, int8_t *q, uint16_t *sx, hipStream_t s)
{
    const dim3 grid((unsigned)M), block(256);
    if (K <= 2048)
        hipLaunchKernelGGL((act_quant_kernel<BF16, 1>), grid, block, 0, s, X, K, q, sx);
    else if (K <= 4096)
        hipLaunchKernelGGL((act_quant_kernel<BF16, 2>), grid, block, 0, s, X, K, q, sx);
    else
        hipLaunchKernelGGL((act_quant_kernel<BF16, 4>), grid, block, 0, s, X, K, q, sx);
}

}  // namespace

hipError_t launch_act_quant(const void *X, bool bf16, int64_t M, int64_t K, int8_t *q,
                            uint16_t *sx, hipStream_t stream)
{
    if (bf16)
        act_quant<true>(X, M, K, q, sx, stream);
    else
        act_quant<false>(X, M, K, q, sx, stream);
    return hipGetLastError();
}

hipError_t launch_quantize(int fmt, const float *W, int64_t N, int64_t K, uint8_t *codes,
                           uint16_t *scales, int *status, hipStream_t stream)
{
    const int64_t n_blocks = N * (K / 32);
    const int64_t threads = n_blocks * 4;
    const int64_t grid = (threads + 255) / 256;
    if (fmt == QL_FMT_INT8)
        hipLaunchKernelGGL(quantize_kernel<QL_FMT_INT8>, dim3((unsigned)grid), dim3(256), 0,
                           stream, W, n_blocks, codes, scales, status);
    else
        hipLaunchKernelGGL(quantize_kernel<QL_FMT_Q4>, dim3((unsigned)grid), dim3(256), 0,
                           stream, W, n_blocks, codes, scales, status);
    return hipGetLastError();
}

}  // namespace qlk
