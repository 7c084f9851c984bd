// Linear forward for few to a few hundred activation rows, in its exact
// per-block form, one launch and no partial sums in memory (bf16 or fp32 X with
// int8 or q4 weights; fp16 weights against the pre-pass's fp16 copy of a bf16
// X):
//
//   Y[m][n] = sum_b s[n][b] * sum_{k in b} X[m][k] * c[n][k]
//
// Why.  At these sizes a layer is a few MB of codes and at most a few GFLOP,
// so what decides is how many of the 256 CUs have work, how much of it is in
// flight, and how many launches there are.  Cutting K into parts over
// workgroups fills the GPU but stores fp32 partials and needs a second
// launch to add them (4 to 6 us each).  Here the 16 wavefronts of a
// workgroup cut K among themselves: KG groups of WN wavefronts own the same
// TM x TN output tile, each its share of every stage's k, and their sums are
// added through LDS in group order at the end.
//
// Shapes (per layer, chosen by kg_plan): TM = 32 or 64 rows, and WN x KG = 4 x
// 4, 2 x 8 or 1 x 16, i.e. TN = 128, 64 or 32 columns; each wavefront owns
// TM x 32 outputs.  One more has 16 columns (16 x 16 x 32 MFMAs), for long
// reductions over few rows: twice the workgroups (a d = 1536 int8 block at 27
// rows 18.5 -> 14.9 us with FFN-down in it).  Sixteen wavefronts
// because one wavefront issues a VALU instruction every ~5 cycles at best
// while a SIMD takes one every 2 to 4 from several.
//
// Memory.  Activations, codes and scales of a stage (256 to 1024 k) go to LDS
// by direct-to-LDS loads of 16 bytes per lane, at least 128 contiguous bytes
// per row, through a ring of NST stages; the loads of a stage go out spread
// over the step before.  Up to 32 rows only the first XR = 8, 16 or 32 are
// staged: the MFMA's other rows repeat them and are never stored.
//
// Contraction.  Per 32-k block and 32 x 32 tile two
// v_mfma_f32_32x32x16_bf16 over k = 32 b + 16 g + 8 h + e (lane group g =
// lane / 32, chunk h, element e), then acc += s * partial in fp32.  The codes
// are converted as signed bytes (q4: nibbles in the high half of a byte, the
// factor 16 taken out of the scale): exact in bf16 and without the offset
// term, and its MFMAs, of the unsigned forms.  With fp32 activations, whose
// other kernel takes the q4 codes as they are, so does this one: 16 times them
// would overflow a block's partial sum at 1/16 of the activations.
//
// Requirements (checked by the host): K % 256 == 0, K < 2^22 (32-bit offsets
// within a tile's fp32 activations or fp16 weights), 16-byte aligned X, codes
// and scales.
#include <algorithm>
#include <type_traits>

#include "dma.h"
#include "epilogue.h"
#include "internal.h"

namespace qlk {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int WAVES = 16, NT = 64 * WAVES;

template <int FMT_, bool XF32_, int XR_, int WN_, int BPW_, int CW_ = 32>
struct KgGeo {
    static constexpr int FMT = FMT_, XR = XR_, WN = WN_, BPW = BPW_;
    static constexpr int CW = CW_;                     // columns per wavefront
    static constexpr bool XF32 = XF32_;
    static constexpr int MI = XR > 32 ? XR / 32 : 1;   // MFMA row blocks
    static constexpr int KG = WAVES / WN;
    static constexpr int TM = XR, TN = CW * WN;
    static constexpr int EB = KG * BPW;                // 32-k blocks per stage
    static constexpr int XRB = EB * (XF32 ? 128 : 64), XCH = XRB / 16;  // activation bytes,
                                                                        // chunks per row
    static constexpr int CRB = FMT == QL_FMT_F16 ? EB * 64 : FMT == QL_FMT_INT8 ? EB * 32 : EB * 16;
    static constexpr int CCH = CRB / 16;
    static constexpr int SCH = FMT == QL_FMT_F16 ? 0 : EB / 8;  // 16-byte scale chunks per column
    static constexpr int XBYTES = XR * XRB, CBYTES = TN * CRB, SBYTES = TN * SCH * 16;
    // loads in units of one wavefront (1 KB); wavefront w takes units w, w +
    // 16, ..., the last ones repeated so that every wavefront counts the same
    static constexpr int XU = XBYTES / 1024, CU = CBYTES / 1024, SU = (SBYTES + 1023) / 1024;
    static constexpr int UNITS = XU + CU + SU, LOADS = (UNITS + WAVES - 1) / WAVES;
    static constexpr int RED = KG * TM * TN * 4;       // the groups' sums at the end
    // two stages ahead where they fit (deeper rings were no faster).  A launch
    // holds the LDS of its largest shape, so that one workgroup is resident per
    // CU (two only of q4's at 9 to 16 rows)
    static constexpr int SLOT = XBYTES + CBYTES + SU * 1024;
    static constexpr int NST = std::min(3, 160 * 1024 / SLOT), RING = NST * SLOT;
    static_assert(NST >= 2, "a stage ahead");
    static constexpr int LDS = RING > RED ? RING : RED;
    static_assert(CW == 32 || (CW == 16 && !XF32 && FMT != QL_FMT_F16 && XR <= 32), "forms built");
    static_assert(EB % 8 == 0 && XBYTES % 1024 == 0 && CBYTES % 1024 == 0, "whole loads");
    static_assert(LDS <= 160 * 1024, "LDS of a CU");
};

// chunk swizzles (physical = logical ^ swizzle): the fragment reads of 16
// consecutive lanes (rows, one logical chunk) fall on distinct banks
__device__ inline int xswz(int row) { return row & 15; }
template <int CCH>
__device__ inline int cswz(int row)
{
    return CCH >= 16 ? row & 15 : (row >> 1) & 7;  // 128-byte rows: two per bank row
}

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
__device__ inline f32x16 mfma_f16(u32x4 a, u32x4 b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, a),
                                                  __builtin_bit_cast(half8, b), c, 0, 0, 0);
}
__device__ inline f32x16 mfma(u32x4 a, u32x4 b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// workgroup p of a layer of G: each XCD (p % 8) takes a contiguous range
__device__ inline int logical_tile(int p, int G)
{
    const int q = G >> 3, r = G & 7;
    const int xcd = p & 7, idx = p >> 3;
    return xcd < r ? xcd * (q + 1) + idx : r * (q + 1) + (xcd - r) * q + idx;
}

__device__ inline float f16_value(uint32_t bits)
{
    return (float)__builtin_bit_cast(_Float16, (uint16_t)bits);
}

// bf16 pair of two fp32 values that bf16 holds exactly
__device__ inline uint32_t bf16_pair(float lo, float hi)
{
    return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
}
__device__ inline float sbyte(uint32_t w, int i) { return (float)((int)(w << (24 - 8 * i)) >> 24); }

// 8 codes (16-k chunk half of a lane) as bf16 pairs in k order
__device__ inline u32x4 cvt_int8(uint32_t w0, uint32_t w1)
{
    return u32x4{bf16_pair(sbyte(w0, 0), sbyte(w0, 1)), bf16_pair(sbyte(w0, 2), sbyte(w0, 3)),
                 bf16_pair(sbyte(w1, 0), sbyte(w1, 1)), bf16_pair(sbyte(w1, 2), sbyte(w1, 3))};
}
// q4: 16 times the codes (nibbles moved to the high half of their bytes,
// read as signed bytes); the scale is divided by 16
__device__ inline u32x4 cvt_q4(uint32_t w)
{
    const uint32_t e = (w << 4) & 0xF0F0F0F0u, o = w & 0xF0F0F0F0u;  // even, odd k
    return u32x4{bf16_pair(sbyte(e, 0), sbyte(o, 0)), bf16_pair(sbyte(e, 1), sbyte(o, 1)),
                 bf16_pair(sbyte(e, 2), sbyte(o, 2)), bf16_pair(sbyte(e, 3), sbyte(o, 3))};
}

// the q4 codes themselves (fp32 activations): each nibble to a signed byte as
// (n ^ 8) - 8, bit 7 of the byte taking the borrow
__device__ inline u32x4 cvt_q4_plain(uint32_t w)
{
    auto bytes = [](uint32_t n) {
        return (((n & 0x0F0F0F0Fu) ^ 0x88888888u) - 0x08080808u) ^ 0x80808080u;
    };
    const uint32_t e = bytes(w), o = bytes(w >> 4);  // even, odd k
    return u32x4{bf16_pair(sbyte(e, 0), sbyte(o, 0)), bf16_pair(sbyte(e, 1), sbyte(o, 1)),
                 bf16_pair(sbyte(e, 2), sbyte(o, 2)), bf16_pair(sbyte(e, 3), sbyte(o, 3))};
}

// 8 fp32 activations as three bf16 planes whose sum they are exactly
// (truncation: 8 + 8 + 8 significant bits)
__device__ inline void split3(u32x4 v0, u32x4 v1, u32x4 &hi, u32x4 &mid, u32x4 &lo)
{
    uint32_t m[8], l[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const uint32_t x = e < 4 ? v0[e] : v1[e - 4];
        const float r = __uint_as_float(x) - __uint_as_float(x & 0xFFFF0000u);
        m[e] = __float_as_uint(r);
        l[e] = __float_as_uint(r - __uint_as_float(m[e] & 0xFFFF0000u));
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const uint32_t a = e < 2 ? v0[2 * e] : v1[2 * e - 4];
        const uint32_t b = e < 2 ? v0[2 * e + 1] : v1[2 * e - 3];
        hi[e] = __builtin_amdgcn_perm(b, a, 0x07060302u);
        mid[e] = __builtin_amdgcn_perm(m[2 * e + 1], m[2 * e], 0x07060302u);
        lo[e] = __builtin_amdgcn_perm(l[2 * e + 1], l[2 * e], 0x07060302u);
    }
}

// One output tile of layer d.
template <class G>
__device__ inline void kg_tile(const LinDesc &d, int tile, uint8_t *ring)
{
    constexpr int FMT = G::FMT, MI = G::MI, XB = G::XF32 ? 4 : 2;
    constexpr bool Q4 = FMT == QL_FMT_Q4, F16 = FMT == QL_FMT_F16;
    const int tm = tile % d.tiles_m, tn = tile / d.tiles_m;
    const int M = d.M, N = d.N, K = d.K, nb = K >> 5;
    const int m0 = tm * G::TM, n0 = tn * G::TN;
    const int crow = Q4 ? K / 2 : F16 ? 2 * K : K;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, g = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = wave / G::WN, wn = (wave % G::WN) * G::CW;

    // this wavefront's loads: per unit a base, a per-lane offset within the
    // stage's first columns, and the bytes a stage advances.  Rows past M and
    // N repeat the last one; chunks past K (a part-filled last stage) the last
    // chunk, and are not used.
    const uint8_t *ub[G::LOADS];
    uint32_t urow[G::LOADS];
    int ucol[G::LOADS], ustep[G::LOADS], ulim[G::LOADS];
    uint32_t udst[G::LOADS];
#pragma unroll
    for (int q = 0; q < G::LOADS; ++q) {
        const int u = min(q * WAVES + wave, G::UNITS - 1);  // wave-uniform
        if (u < G::XU) {
            const int slot = u * 64 + lane, row = slot / G::XCH;
            ub[q] = reinterpret_cast<const uint8_t *>(d.X) + (int64_t)m0 * K * XB;
            urow[q] = (uint32_t)((min(m0 + row, M - 1) - m0) * K * XB);
            ucol[q] = ((slot % G::XCH) ^ xswz(row)) * 16;
            ustep[q] = G::XRB;
            ulim[q] = K * XB - 16;
            udst[q] = u * 1024;
        } else if (u < G::XU + G::CU) {
            const int slot = (u - G::XU) * 64 + lane, row = slot / G::CCH;
            ub[q] = d.codes + (int64_t)n0 * crow;
            urow[q] = (uint32_t)((min(n0 + row, N - 1) - n0) * crow);
            ucol[q] = ((slot % G::CCH) ^ cswz<G::CCH>(row)) * 16;
            ustep[q] = G::CRB;
            ulim[q] = crow - 16;
            udst[q] = u * 1024;
        } else if constexpr (!F16) {
            // scales: chunk-major, [SCH][TN] of 16 bytes
            const int slot = ((u - G::XU - G::CU) * 64 + lane) % (G::TN * G::SCH);
            const int row = slot % G::TN;
            ub[q] = reinterpret_cast<const uint8_t *>(d.scales) + (int64_t)n0 * nb * 2;
            urow[q] = (uint32_t)((min(n0 + row, N - 1) - n0) * nb * 2);
            ucol[q] = (slot / G::TN) * 16;
            ustep[q] = G::SCH * 16;
            ulim[q] = nb * 2 - 16;
            udst[q] = u * 1024;
        }
    }
    const int iters = (nb + G::EB - 1) / G::EB;
    auto issue = [&](int it, int q) {
        dma_load16(ub[q], urow[q] + (uint32_t)min(it * ustep[q] + ucol[q], ulim[q]),
                   dma_lds(ring + (it % G::NST) * G::SLOT) + udst[q]);
    };
#pragma unroll
    for (int it = 0; it < G::NST - 1; ++it)
        if (it < iters)
#pragma unroll
            for (int q = 0; q < G::LOADS; ++q)
                issue(it, q);

    // accumulator registers that hold staged rows: 8 (r / 4) + 4 g + r % 4
    constexpr int AR = G::XR < 32 ? G::XR / 2 : 16;
    f32x16 acc[MI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
        acc[i] = f32x16{};
    // 16 columns: 16 x 16 tiles, register r of lane l holding row 16 i + 4 (l /
    // 16) + r, column l % 16
    constexpr bool C16 = G::CW == 16;
    constexpr int MI16 = (G::XR + 15) / 16;
    f32x4 acc16[MI16];
#pragma unroll
    for (int i = 0; i < MI16; ++i)
        acc16[i] = f32x4{};
    const int l16 = lane & 15, lg = lane >> 4;

    auto step = [&](int it, auto refill) {
        constexpr bool REFILL = decltype(refill)::value;
        // every LDS read of the previous stage has completed; this one landed
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if constexpr (REFILL)
            __builtin_amdgcn_s_waitcnt(dma_vmcnt((G::NST - 2) * G::LOADS));
        else
            dma_wait<G::LOADS, G::NST - 2>(iters - 1 - it);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");  // no LDS read moves above the barrier
        const uint8_t *const st = ring + (it % G::NST) * G::SLOT;
#pragma unroll
        for (int u = 0; u < G::BPW; ++u) {
            const int b = kg * G::BPW + u;  // block of the stage
            // past K (the last stage only, which refills nothing)
            if constexpr (!REFILL)
                if (it * G::EB + b >= nb)
                    continue;
            if constexpr (REFILL)
#pragma unroll
                for (int q = u; q < G::LOADS; q += G::BPW)
                    issue(it + G::NST - 1, q);
            const int wr = wn + (C16 ? l16 : l32);
            const uint8_t *const wrow = st + G::XBYTES + wr * G::CRB;
            float s = 1.0f;
            u32x4 wv[2];
            if constexpr (C16) {
                const uint32_t sw = *reinterpret_cast<const uint16_t *>(
                    st + G::XBYTES + G::CBYTES + ((b / 8) * G::TN + wr) * 16 + (b % 8) * 2);
                s = f16_value(sw) * (Q4 ? 0.0625f : 1.0f);  // exact
                dma_pin(s);
                // the lane's 8 codes of the block: k = 32 b + 8 (lane / 16) + e
                if constexpr (Q4) {
                    wv[0] = cvt_q4(*reinterpret_cast<const uint32_t *>(
                        wrow + (b ^ cswz<G::CCH>(wr)) * 16 + 4 * lg));
                } else {
                    const u32x2 c = *reinterpret_cast<const u32x2 *>(
                        wrow + ((2 * b + (lg >> 1)) ^ cswz<G::CCH>(wr)) * 16 + 8 * (lg & 1));
                    wv[0] = cvt_int8(c[0], c[1]);
                }
#pragma unroll
                for (int i = 0; i < MI16; ++i) {
                    const int xr = 16 * i + (l16 & (G::XR < 16 ? G::XR - 1 : 15));
                    const u32x4 x = *reinterpret_cast<const u32x4 *>(
                        st + xr * G::XRB + ((4 * b + lg) ^ xswz(xr)) * 16);
                    const f32x4 p = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        __builtin_bit_cast(bf16x8, x), __builtin_bit_cast(bf16x8, wv[0]), f32x4{},
                        0, 0, 0);
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        acc16[i][r] = __builtin_fmaf(s, p[r], acc16[i][r]);
                }
                continue;
            }
            if constexpr (F16) {
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    wv[h] = *reinterpret_cast<const u32x4 *>(
                        wrow + ((4 * b + 2 * g + h) ^ cswz<G::CCH>(wr)) * 16);
            } else {
                const uint32_t sw = *reinterpret_cast<const uint16_t *>(
                    st + G::XBYTES + G::CBYTES + ((b / 8) * G::TN + wr) * 16 + (b % 8) * 2);
                s = f16_value(sw) * (Q4 && !G::XF32 ? 0.0625f : 1.0f);  // exact
                dma_pin(s);
                // the lane's codes of the block: 16 (int8) or 8 (q4) bytes
                if constexpr (Q4) {
                    const u32x2 c = *reinterpret_cast<const u32x2 *>(
                        wrow + (b ^ cswz<G::CCH>(wr)) * 16 + 8 * g);
                    wv[0] = G::XF32 ? cvt_q4_plain(c[0]) : cvt_q4(c[0]);
                    wv[1] = G::XF32 ? cvt_q4_plain(c[1]) : cvt_q4(c[1]);
                } else {
                    const u32x4 c = *reinterpret_cast<const u32x4 *>(
                        wrow + ((2 * b + g) ^ cswz<G::CCH>(wr)) * 16);
                    wv[0] = cvt_int8(c[0], c[1]);
                    wv[1] = cvt_int8(c[2], c[3]);
                }
            }
            f32x16 p[MI];
#pragma unroll
            for (int i = 0; i < MI; ++i) {
                const int xr = 32 * i + (l32 & (G::XR < 32 ? G::XR - 1 : 31));
                const uint8_t *const xrow = st + xr * G::XRB;
                if constexpr (G::XF32) {
                    u32x4 hi[2], mid[2], lo[2];
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const int lc = 8 * b + 4 * g + 2 * h;
                        split3(*reinterpret_cast<const u32x4 *>(xrow + (lc ^ xswz(xr)) * 16),
                               *reinterpret_cast<const u32x4 *>(xrow + ((lc + 1) ^ xswz(xr)) * 16),
                               hi[h], mid[h], lo[h]);
                    }
                    p[i] = mfma(lo[0], wv[0], f32x16{});
                    p[i] = mfma(lo[1], wv[1], p[i]);
                    p[i] = mfma(mid[0], wv[0], p[i]);
                    p[i] = mfma(mid[1], wv[1], p[i]);
                    p[i] = mfma(hi[0], wv[0], p[i]);
                    p[i] = mfma(hi[1], wv[1], p[i]);
                } else {
                    u32x4 a[2];
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        a[h] = *reinterpret_cast<const u32x4 *>(
                            xrow + ((4 * b + 2 * g + h) ^ xswz(xr)) * 16);
                    if constexpr (F16) {
                        acc[i] = mfma_f16(a[0], wv[0], acc[i]);
                        acc[i] = mfma_f16(a[1], wv[1], acc[i]);
                    } else {
                        p[i] = mfma(a[0], wv[0], f32x16{});
                        p[i] = mfma(a[1], wv[1], p[i]);
                    }
                }
            }
            if constexpr (!F16)
#pragma unroll
                for (int i = 0; i < MI; ++i)
#pragma unroll
                    for (int r = 0; r < AR; ++r)
                        acc[i][r] = __builtin_fmaf(s, p[i][r], acc[i][r]);
        }
    };
    int it = 0;
#pragma unroll 1
    for (; it + G::NST - 1 < iters; ++it)
        step(it, std::true_type{});
#pragma unroll 1
    for (; it < iters; ++it)
        step(it, std::false_type{});

    // The groups' sums as rows in LDS (every stage issued has been waited
    // for and, behind the barrier, read), then every thread adds and stores
    // groups of four columns.
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    float *const red = reinterpret_cast<float *>(ring);
    if constexpr (C16) {
#pragma unroll
        for (int i = 0; i < MI16; ++i)
            if (16 * i + 4 * lg < G::TM)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    red[(kg * G::TM + 16 * i + 4 * lg + r) * G::TN + wn + l16] = acc16[i][r];
    }
#pragma unroll
    for (int i = 0; i < MI && !C16; ++i)
#pragma unroll
        for (int r = 0; r < AR; ++r)
            red[(kg * G::TM + 32 * i + 8 * (r >> 2) + 4 * g + (r & 3)) * G::TN + wn + l32] =
                acc[i][r];
    __syncthreads();
    const bool vec = epi_vec_ok(d.ep, d.Y, N);
#pragma unroll 1
    for (int q = tid; q < G::TM * G::TN / 4; q += NT) {
        const int m = m0 + q / (G::TN / 4), n = n0 + 4 * (q % (G::TN / 4));
        if (m >= M || n >= N)
            continue;
        const f32x4 *const src = reinterpret_cast<const f32x4 *>(red) + q;
        f32x4 v = src[0];
#pragma unroll
        for (int k = 1; k < G::KG; ++k)
            v += src[k * (G::TM * G::TN / 4)];
        if constexpr (F16) {  // the activations' row shift
            const int e = d.xexp[m];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                v[k] = __builtin_ldexpf(v[k], e);
        }
        const int64_t idx = (int64_t)m * N + n;
        if (vec) {
            epi_store4(d.ep, d.Y, idx, n, v, false);
        } else {
#pragma unroll 1
            for (int e = 0; e < 4 && n + e < N; ++e)
                epi_store(d.ep, d.Y, idx + e, n + e, v[e]);
        }
    }
}

// The shapes a launch may mix.  bf16 X and quantized weights: XR = 8, 16 or
// 32 for launches of at most that many rows and 64 above.
template <int FMT, int XR>
struct KgShapes {
    static constexpr bool I8 = FMT == QL_FMT_INT8;
    static constexpr int XR1 = XR < 32 ? XR : 32;
    // up to 8 rows a stage is small: twice the k per stage, half the barriers
    static constexpr bool FEW = XR <= 8;
    using R1W4 = KgGeo<FMT, false, XR1, 4, FEW ? 4 : 2>;
    using R1W2 = KgGeo<FMT, false, XR1, 2, FEW ? 2 : 1>;
    using R1W1 = KgGeo<FMT, false, XR1, 1, FEW ? 2 : 1>;
    using R1C16 = KgGeo<FMT, false, XR1, 1, FEW ? 2 : 1, 16>;
    using R2W4 = KgGeo<FMT, false, 64, 4, 2>;
    using R2W2 = KgGeo<FMT, false, 64, 2, 1>;
    // (16 columns of q4 at up to 16 rows cost more per workgroup than 32 and
    // there are twice as many: no plan takes them)
    static constexpr bool R2 = XR > 32, R2_W4 = R2, C16 = I8 || XR > 16;
};
// fp16 weights (X the fp16 copy of the pre-pass)
template <int XR>
struct KgShapes<QL_FMT_F16, XR> {
    using R1W4 = KgGeo<QL_FMT_F16, false, 32, 4, 2>;
    using R1W2 = KgGeo<QL_FMT_F16, false, 32, 2, 1>;
    using R1W1 = KgGeo<QL_FMT_F16, false, 32, 1, 1>;
    using R2W2 = KgGeo<QL_FMT_F16, false, 64, 2, 1>;
    using R2W4 = R2W2;
    using R1C16 = R1W1;
    static constexpr bool R2 = true, R2_W4 = false, C16 = false;
};
// fp32 X: row tiles of 16 and 32 (a stage of 64 fp32 rows leaves no room for
// a second one)
template <int FMT>
struct KgShapesF32 {
    using R1W4 = KgGeo<FMT, true, 32, 4, 2>;
    using R1W2 = KgGeo<FMT, true, 32, 2, 1>;
    using R1W1 = KgGeo<FMT, true, 16, 1, 1>;
    using R2W2 = KgGeo<FMT, true, 16, 2, 1>;
    using R2W4 = R2W2;
    using R1C16 = R1W1;
    static constexpr bool R2 = true, R2_W4 = false, C16 = false;
};

template <class S>
constexpr int kg_lds()
{
    int v = std::max(S::R1W4::LDS, std::max(S::R1W2::LDS, S::R1W1::LDS));
    if constexpr (S::R2)
        v = std::max(v, S::R2W2::LDS);
    if constexpr (S::R2_W4)
        v = std::max(v, S::R2W4::LDS);
    if constexpr (S::C16)
        v = std::max(v, S::R1C16::LDS);
    return v;
}

template <class S>
__global__ __launch_bounds__(NT, 4) void qgemm_kg_kernel(const GroupArgs args)
{
    __shared__ __align__(16) uint8_t ring[kg_lds<S>()];
    const int p = (int)blockIdx.x;
    LinDesc d = args.d[0];
    int end = args.total_tiles;
#pragma unroll
    for (int t = 1; t < QL_MAX_GROUP; ++t) {
        if (t < args.n && p >= args.d[t].tile_begin)
            d = args.d[t];
        if (t < args.n && p < args.d[t].tile_begin && end == args.total_tiles)
            end = args.d[t].tile_begin;
    }
    const int tile = logical_tile(p - d.tile_begin, end - d.tile_begin);
    switch (d.psteps) {  // shape (the host's plan)
    case KG_R1W1:
        kg_tile<typename S::R1W1>(d, tile, ring);
        break;
    case KG_R1W2:
        kg_tile<typename S::R1W2>(d, tile, ring);
        break;
    case KG_R1W4:
        kg_tile<typename S::R1W4>(d, tile, ring);
        break;
    case KG_R1C16:
        if constexpr (S::C16)
            kg_tile<typename S::R1C16>(d, tile, ring);
        break;
    case KG_R2W2:
        if constexpr (S::R2)
            kg_tile<typename S::R2W2>(d, tile, ring);
        break;
    default:
        if constexpr (S::R2_W4)
            kg_tile<typename S::R2W4>(d, tile, ring);
    }
}

template <class S>
hipError_t launch_shapes(const GroupArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL(qgemm_kg_kernel<S>, dim3((unsigned)a.total_tiles), dim3(NT), 0, s, a);
    return hipGetLastError();
}

template <int FMT>
hipError_t launch_fmt(bool xf32, int maxM, const GroupArgs &a, hipStream_t s)
{
    if (xf32)
        return launch_shapes<KgShapesF32<FMT>>(a, s);
    return maxM > 32   ? launch_shapes<KgShapes<FMT, 64>>(a, s)
           : maxM > 16 ? launch_shapes<KgShapes<FMT, 32>>(a, s)
           : maxM > 8  ? launch_shapes<KgShapes<FMT, 16>>(a, s)
                       : launch_shapes<KgShapes<FMT, 8>>(a, s);
}

// rows and columns of a shape's tile
template <class S>
KgTile tile_of(int shape)
{
    switch (shape) {
    case KG_R1W1: return KgTile{S::R1W1::TM, S::R1W1::TN};
    case KG_R1W2: return KgTile{S::R1W2::TM, S::R1W2::TN};
    case KG_R1W4: return KgTile{S::R1W4::TM, S::R1W4::TN};
    case KG_R1C16: return S::C16 ? KgTile{S::R1C16::TM, S::R1C16::TN} : KgTile{0, 0};
    case KG_R2W2: return S::R2 ? KgTile{S::R2W2::TM, S::R2W2::TN} : KgTile{0, 0};
    default: return S::R2_W4 ? KgTile{S::R2W4::TM, S::R2W4::TN} : KgTile{0, 0};
    }
}

template <int FMT>
KgTile tile_fmt(bool xf32, int64_t maxM, int shape)
{
    if (xf32)
        return tile_of<KgShapesF32<FMT>>(shape);
    return maxM > 32   ? tile_of<KgShapes<FMT, 64>>(shape)
           : maxM > 16 ? tile_of<KgShapes<FMT, 32>>(shape)
           : maxM > 8  ? tile_of<KgShapes<FMT, 16>>(shape)
                       : tile_of<KgShapes<FMT, 8>>(shape);
}

}  // namespace

KgTile kg_tile_shape(int fmt, bool xf32, int64_t maxM, int shape)
{
    if (fmt == QL_FMT_F16)
        return tile_of<KgShapes<QL_FMT_F16, 64>>(shape);
    return fmt == QL_FMT_INT8 ? tile_fmt<QL_FMT_INT8>(xf32, maxM, shape)
                              : tile_fmt<QL_FMT_Q4>(xf32, maxM, shape);
}

hipError_t launch_qgemm_kg(int fmt, bool xf32, int maxM, const GroupArgs &args, hipStream_t stream)
{
    if (fmt == QL_FMT_F16)
        return launch_shapes<KgShapes<QL_FMT_F16, 64>>(args, stream);
    return fmt == QL_FMT_INT8 ? launch_fmt<QL_FMT_INT8>(xf32, maxM, args, stream)
                              : launch_fmt<QL_FMT_Q4>(xf32, maxM, args, stream);
}

}  // namespace qlk
