// W8A8 forward: per-token int8 activations against int8 block-quantized
// weights on the int8 matrix cores.
//
// Paper (Methodology, the 8-bit-arithmetic mode of the runtime; Table II):
// activations are quantized alongside the weights and the products run in
// 8-bit integers.  With per-token activation scales s_x[m] and the weights'
// per-block scales s[n][b]:
//
//   Y[m][n] = s_x[m] * sum_b s[n][b] * D_b[m][n],
//   D_b[m][n] = sum_{k in block b} q[m][k] * c[n][k]      (exact, int32)
//
// Each 32 x 32 output tile of a 32-k block is one v_mfma_i32_32x32x32_i8
// (exact), converted and folded into an fp32 accumulator with one FMA per
// output (scale of the lane's column); s_x[m] and the layer epilogue are
// applied at the store.  The per-block rescale is what bounds this path:
// 16 outputs per lane per MFMA cost two VALU instructions each (64 issue
// cycles against the MFMA's 32), so a kernel can at best keep every SIMD's
// VALU issuing: M N K / 32 * 2 lane operations.
//
// Two kernels.  qgemm_w8a8_pipe_kernel takes K % 64 == 0 with 4-byte aligned
// scales; qgemm_w8a8_kernel the rest (an odd number of blocks, scales at odd
// 2-byte addresses).
#include "dma.h"
#include "epilogue.h"
#include "internal.h"
#include <type_traits>

namespace qlk {
namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x16 __attribute__((ext_vector_type(16)));

constexpr int BM = 128, BN = 128, BK = 64;
constexpr int THREADS = 256;
constexpr int ROW = 80;                    // LDS bytes per tile row (64 + 16)
constexpr int TILE = BM * ROW;             // one operand tile
constexpr int STAGE = 2 * TILE + 2 * BN * 4;  // X tile, W tile, scales [2][BN] fp32
constexpr int GROUP_M = 8;                 // row tiles that share a column sweep
static_assert(BM == BN, "one chunk mapping serves both operand tiles");

__device__ inline float f16_value(uint16_t bits)
{
    return (float)__builtin_bit_cast(_Float16, bits);
}

// Workgroup p runs on XCD p % 8; give each XCD a contiguous range of the T
// tiles so that neighbouring tiles share an L2.
__device__ inline int xcd_tile(int p, int T)
{
    const int q = T >> 3, r = T & 7;
    const int xcd = p & 7, idx = p >> 3;
    return xcd < r ? xcd * (q + 1) + idx : r * (q + 1) + (xcd - r) * q + idx;
}

// General kernel: 128 x 128 outputs per workgroup of 4 wavefronts (64 x 64
// each, 2 x 2 MFMA tiles), K in stages of 64 (two blocks) double-buffered in
// LDS through registers; rows padded to 80 bytes so that the 32 rows an
// operand read touches spread over the LDS banks.
__global__ __launch_bounds__(THREADS, 2) void qgemm_w8a8_kernel(const W8Args a)
{
    __shared__ __align__(16) uint8_t lds[2 * STAGE];
    const int T = a.tiles_m * a.tiles_n;
    const int tile = xcd_tile((int)blockIdx.x, T);
    const int per_group = GROUP_M * a.tiles_n;
    const int first_m = (tile / per_group) * GROUP_M;
    const int gsz = min(a.tiles_m - first_m, GROUP_M);
    const int within = tile % per_group;
    const int m0 = (first_m + within % gsz) * BM, n0 = (within / gsz) * BN;

    const int M = a.M, N = a.N, K = a.K, nb = K / 32;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;  // the wave's 64 x 64
    const int l32 = lane & 31, hi = lane >> 5;

    // staging: thread t moves 16-byte chunks c = t and t + 256 of each
    // operand tile (row c / 4, bytes 16 (c % 4) of the stage's 64) and the
    // scale of column t % 128, block t / 128 of the stage
    int crow[2], ccol[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        crow[i] = (tid + THREADS * i) >> 2;
        ccol[i] = 16 * ((tid + THREADS * i) & 3);
    }
    const int scol = tid & (BN - 1), sblk = tid >> 7;
    i32x4 px[2], pw[2];
    float ps;
    auto fetch = [&](int s) {
        const int k0 = s * BK;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int k = k0 + ccol[i];
            const int mr = m0 + crow[i], nr = n0 + crow[i];
            px[i] = mr < M && k < K
                        ? *reinterpret_cast<const i32x4 *>(a.qx + (int64_t)mr * K + k)
                        : i32x4{0, 0, 0, 0};
            pw[i] = nr < N && k < K
                        ? *reinterpret_cast<const i32x4 *>(a.codes + (int64_t)nr * K + k)
                        : i32x4{0, 0, 0, 0};
        }
        const int b = 2 * s + sblk, n = n0 + scol;
        ps = n < N && b < nb ? f16_value(a.scales[(int64_t)n * nb + b]) : 0.0f;
    };
    auto put = [&](int buf) {
        uint8_t *st = lds + buf * STAGE;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            *reinterpret_cast<i32x4 *>(st + crow[i] * ROW + ccol[i]) = px[i];
            *reinterpret_cast<i32x4 *>(st + TILE + crow[i] * ROW + ccol[i]) = pw[i];
        }
        reinterpret_cast<float *>(st + 2 * TILE)[sblk * BN + scol] = ps;
    };

    float acc[2][2][16];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                acc[i][j][r] = 0.0f;

    const int nsteps = (K + BK - 1) / BK;
    fetch(0);
    put(0);
    __syncthreads();
    for (int s = 0; s < nsteps; ++s) {
        if (s + 1 < nsteps)
            fetch(s + 1);
        const uint8_t *st = lds + (s & 1) * STAGE;
        const float *sc = reinterpret_cast<const float *>(st + 2 * TILE);
#pragma unroll
        for (int blk = 0; blk < 2; ++blk) {
            // lane (l32, hi) holds row l32 of the A tile and column l32 of
            // the B tile, k = 16 hi .. 16 hi + 15 of the block
            i32x4 av[2], bv[2];
            float sw[2];
#pragma unroll
            for (int i = 0; i < 2; ++i)
                av[i] = *reinterpret_cast<const i32x4 *>(st + (wm + 32 * i + l32) * ROW +
                                                         32 * blk + 16 * hi);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                bv[j] = *reinterpret_cast<const i32x4 *>(st + TILE + (wn + 32 * j + l32) * ROW +
                                                         32 * blk + 16 * hi);
                sw[j] = sc[blk * BN + wn + 32 * j + l32];
            }
            i32x16 dv[2][2];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    dv[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(
                        av[i], bv[j], i32x16{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0},
                        0, 0, 0);
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        acc[i][j][r] = __builtin_fmaf(sw[j], (float)dv[i][j][r], acc[i][j][r]);
        }
        if (s + 1 < nsteps)
            put((s + 1) & 1);
        __syncthreads();
    }

    // output (row 8 (r / 4) + 4 hi + r % 4, column l32 of each 32 x 32 tile):
    // times the row's activation scale, then the layer epilogue
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int m = m0 + wm + 32 * i + 8 * (r >> 2) + 4 * hi + (r & 3);
            if (m >= M)
                continue;
            const float sxm = f16_value(a.sx[m]);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int n = n0 + wn + 32 * j + l32;
                if (n < N)
                    epi_store(a.ep, a.Y, (int64_t)m * N + n, n, sxm * acc[i][j][r]);
            }
        }
}

// Pipelined kernel (K % 64 == 0, K < 2^23, scales 4-byte aligned).
//
// A workgroup is KG groups of WM x WN wavefronts; every wavefront owns 64 x
// (32 NJ) outputs (2 x NJ MFMA tiles), the groups the same (64 WM) x (32 NJ
// WN) output tile over interleaved 64-k steps, and their fp32 sums are added
// through LDS in group order at the end.  K groups are how a product with
// few output tiles (a 1536-wide layer at 1290 tokens has 132 of 128 x 128)
// still gives every SIMD four wavefronts without partial sums in memory.
//
// Four wavefronts per SIMD because one wavefront issues a VALU instruction
// every ~5 cycles at best (2.0 to 2.2 ns measured), while the SIMD takes an fp32
// add or FMA from several every 2 (1.02 to 1.06 ns; v_fma_mix_f32 and the
// int-to-float conversion take 4, 1.83 ns: hence the explicit fp32 scales and
// the seeded accumulators below).
//
// Activations, codes and scales go to LDS by direct-to-LDS loads through a
// ring of NST stages of SB steps per group: at least 128 contiguous bytes of
// every row (64-byte rows took 10-20% longer: the traffic from L2, 6-8 TB/s
// here, is the second bound).  A stage's loads go out one behind each MFMA:
// issued together they hold every wavefront up at the top of the step.
// Within a step the MFMA of a tile is issued before the 32 rescale
// instructions of the tile before it, so that the VALU always has work.
template <int NJ_, int WM_, int WN_, int KG_, int SB_, int NST_, int OCC_>
struct PipeGeo {
    static constexpr int NJ = NJ_, WM = WM_, WN = WN_, KG = KG_, SB = SB_, NST = NST_, OCC = OCC_;
    static constexpr int NT = 64 * WM * WN * KG;        // threads of a workgroup
    static constexpr int TM = 64 * WM, TN = 32 * NJ * WN;  // output tile
    static constexpr int NS = KG * SB;                  // 64-k steps per stage
    static constexpr int RB = 64 * NS, CH = RB / 16;    // bytes and chunks per row and stage
    static constexpr int XB = TM * RB, WB = TN * RB;    // operand bytes per stage
    static constexpr int XL = XB / 16 / NT, WL = WB / 16 / NT;
    static constexpr int SL = (TN * NS + NT - 1) / NT;  // scale loads (4 bytes each)
    static constexpr int LOADS = XL + WL + SL;          // per thread and stage
    static constexpr int STAGE = XB + WB + SL * NT * 4;
    static constexpr int RED = KG > 1 ? KG * TM * TN * 4 : NT / 64 * 4096;  // output staging
    static constexpr int LDS = NST * STAGE > RED ? NST * STAGE : RED;
    static_assert(XB % (16 * NT) == 0 && WB % (16 * NT) == 0, "whole loads per thread");
    static_assert(LDS <= 160 * 1024, "LDS of a CU");
};

// 16-byte chunk swizzle of a row of CH chunks: the fragment reads of 16
// consecutive lanes (rows, one logical chunk) fall on distinct banks
template <int CH>
__device__ inline int row_swz(int row)
{
    return CH >= 16 ? row & 15
         : CH == 8  ? (row & 7) ^ ((row >> 3) & 1)
                    : ((row >> 1) ^ (row >> 3)) & 3;
}

template <class G>
__global__ __launch_bounds__(G::NT, G::OCC) void qgemm_w8a8_pipe_kernel(const W8Args a)
{
    __shared__ __align__(16) uint8_t ring[G::LDS];
    const int T = a.tiles_m * a.tiles_n;
    const int tile = xcd_tile((int)blockIdx.x, T);
    const int per_group = GROUP_M * a.tiles_n;
    const int first_m = (tile / per_group) * GROUP_M;
    const int gsz = min(a.tiles_m - first_m, GROUP_M);
    const int within = tile % per_group;
    const int m0 = (first_m + within % gsz) * G::TM, n0 = (within / gsz) * G::TN;

    const int M = a.M, N = a.N, K = a.K, nb = K / 32;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hi = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = wave / (G::WM * G::WN), gw = wave % (G::WM * G::WN);
    const int wm = (gw / G::WN) * 64, wn = (gw % G::WN) * 32 * G::NJ;

    const uint8_t *const xb = reinterpret_cast<const uint8_t *>(a.qx) + (int64_t)m0 * K;
    const uint8_t *const cb = reinterpret_cast<const uint8_t *>(a.codes) + (int64_t)n0 * K;
    const uint8_t *const sb = reinterpret_cast<const uint8_t *>(a.scales) + (int64_t)n0 * nb * 2;
    // loads: slot r * NT + tid holds chunk (slot % CH) ^ swizzle of row slot
    // / CH; rows past the edge repeat the last one (their outputs are never
    // stored), chunks past K the last one (their scales are taken as 0)
    uint32_t xrow[G::XL], wrow[G::WL], srow[G::SL];
    int xk[G::XL], wk[G::WL], sk[G::SL];
#pragma unroll
    for (int r = 0; r < G::XL; ++r) {
        const int slot = r * G::NT + tid, row = slot / G::CH;
        xrow[r] = (uint32_t)((min(m0 + row, M - 1) - m0) * K);
        xk[r] = ((slot % G::CH) ^ row_swz<G::CH>(row)) * 16;
    }
#pragma unroll
    for (int r = 0; r < G::WL; ++r) {
        const int slot = r * G::NT + tid, row = slot / G::CH;
        wrow[r] = (uint32_t)((min(n0 + row, N - 1) - n0) * K);
        wk[r] = ((slot % G::CH) ^ row_swz<G::CH>(row)) * 16;
    }
#pragma unroll
    for (int r = 0; r < G::SL; ++r) {
        const int slot = (r * G::NT + tid) % (G::TN * G::NS);
        srow[r] = (uint32_t)((min(n0 + slot / G::NS, N - 1) - n0) * nb * 2);
        sk[r] = (slot % G::NS) * 4;
    }

    const int steps = K / 64, iters = (steps + G::NS - 1) / G::NS;
    // the q-th load (of LOADS) of iteration it
    auto issue = [&](int it, int q) {
        const uint32_t base = dma_lds(ring + (it % G::NST) * G::STAGE);
        if (q < G::XL)
            dma_load16(xb, xrow[q] + (uint32_t)min(it * G::RB + xk[q], K - 16),
                       base + (q * G::NT + wave * 64) * 16);
        else if (q < G::XL + G::WL)
            dma_load16(cb, wrow[q - G::XL] + (uint32_t)min(it * G::RB + wk[q - G::XL], K - 16),
                       base + G::XB + ((q - G::XL) * G::NT + wave * 64) * 16);
        else
            dma_load4(sb,
                      srow[q - G::XL - G::WL] +
                          (uint32_t)min(it * G::NS * 4 + sk[q - G::XL - G::WL], (steps - 1) * 4),
                      base + G::XB + G::WB + ((q - G::XL - G::WL) * G::NT + wave * 64) * 4);
    };
#pragma unroll
    for (int it = 0; it < G::NST - 1; ++it)
        if (it < iters)
#pragma unroll
            for (int q = 0; q < G::LOADS; ++q)
                issue(it, q);

    float acc[2][G::NJ][16];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < G::NJ; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                acc[i][j][r] = 0.0f;
    constexpr int TT = 2 * G::NJ;  // MFMA tiles of a block
    // Every MFMA accumulates onto the bit pattern of 1.5 * 2^23: the sum S
    // (|S| <= 32 * 128 * 128 < 2^22) then reads as the float 1.5 * 2^23 + S,
    // and one exact subtraction converts it (v_cvt_f32_i32 issues at a
    // quarter of that rate).  The seed is opaque to the compiler so that it
    // stays in registers instead of being rebuilt for each MFMA.
    constexpr int SEED = 0x4B400000;
    constexpr float SEEDF = 12582912.0f;
    i32x16 seed = {SEED, SEED, SEED, SEED, SEED, SEED, SEED, SEED,
                   SEED, SEED, SEED, SEED, SEED, SEED, SEED, SEED};
    dma_pin(seed);
    // the tile whose rescale runs behind the next tile's MFMA
    i32x16 pend = seed;
    float pend_s = 0.0f;

    // One iteration; REFILL: a stage NST - 1 ahead is left to load (a
    // compile-time condition, so that the step stays one basic block and the
    // compiler keeps the order written here).
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
        // the slot of the previous stage is free: its refill goes out one
        // load behind each MFMA (together they would hold the wavefronts up
        // at the top of the step, the address unit taking 16 to 64 cycles each)
        const uint8_t *const st = ring + (it % G::NST) * G::STAGE;
        // blocks 0 .. 2 SB - 1 of the group's steps of the stage
        constexpr int NB = 2 * G::SB;
        float sc[NB][G::NJ];
#pragma unroll
        for (int u = 0; u < G::SB; ++u) {
            const int sub = kg * G::SB + u;
            const bool live = it * G::NS + sub < steps;
#pragma unroll
            for (int j = 0; j < G::NJ; ++j) {
                uint32_t w = *reinterpret_cast<const uint32_t *>(
                    st + G::XB + G::WB + ((wn + 32 * j + l32) * G::NS + sub) * 4);
                w = live ? w : 0u;
                sc[2 * u][j] = f16_value((uint16_t)(w & 0xFFFFu));
                sc[2 * u + 1][j] = f16_value((uint16_t)(w >> 16));
                dma_pin(sc[2 * u][j]);
                dma_pin(sc[2 * u + 1][j]);
            }
        }
        // operands of block blk, two blocks alternating
        i32x4 av[2][2], bv[2][G::NJ];
        auto read = [&](int blk) {
            const int lc = 4 * (kg * G::SB + blk / 2) + 2 * (blk & 1) + hi;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int xr = wm + 32 * i + l32;
                av[blk & 1][i] = *reinterpret_cast<const i32x4 *>(
                    st + xr * G::RB + (lc ^ row_swz<G::CH>(xr)) * 16);
            }
#pragma unroll
            for (int j = 0; j < G::NJ; ++j) {
                const int wr = wn + 32 * j + l32;
                bv[blk & 1][j] = *reinterpret_cast<const i32x4 *>(
                    st + G::XB + wr * G::RB + (lc ^ row_swz<G::CH>(wr)) * 16);
            }
        };
        read(0);
#pragma unroll
        for (int blk = 0; blk < NB; ++blk)
#pragma unroll
            for (int t = 0; t < TT; ++t) {
                const int i = t / G::NJ, j = t % G::NJ;
                i32x16 d = __builtin_amdgcn_mfma_i32_32x32x32_i8(av[blk & 1][i], bv[blk & 1][j],
                                                                 seed, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (blk + 1 < NB && t == 0)
                    read(blk + 1);
                if constexpr (REFILL)
#pragma unroll
                    for (int q = blk * TT + t; q < G::LOADS; q += NB * TT)
                        issue(it + G::NST - 1, q);
                // the tile before this one (the previous block's last for t = 0)
                const int pt = (t + TT - 1) % TT, pi = pt / G::NJ, pj = pt % G::NJ;
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    acc[pi][pj][r] = __builtin_fmaf(pend_s, __int_as_float(pend[r]) - SEEDF,
                                                    acc[pi][pj][r]);
                pend = d;
                pend_s = sc[blk][j];
                __builtin_amdgcn_sched_barrier(0);
            }
    };
    int it = 0;
#pragma unroll 1
    for (; it + G::NST - 1 < iters; ++it)
        step(it, std::true_type{});
#pragma unroll 1
    for (; it < iters; ++it)
        step(it, std::false_type{});
#pragma unroll
    for (int r = 0; r < 16; ++r)
        acc[1][G::NJ - 1][r] = __builtin_fmaf(pend_s, __int_as_float(pend[r]) - SEEDF,
                                              acc[1][G::NJ - 1][r]);

    // Output: row 8 (r / 4) + 4 hi + r % 4, column l32 of each 32 x 32 tile.
    // The K groups' tiles go to LDS as rows (the ring is free behind the
    // barrier: every stage issued has been waited for and read), and every
    // thread sums and stores groups of four columns.  One group: each
    // wavefront turns one 32 x 32 tile at a time in a patch of its own.
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    const bool vec = epi_vec_ok(a.ep, a.Y, N);
    auto store4 = [&](int m, int n, f32x4 v) {
        if (m >= M || n >= N)
            return;
        const float sxm = f16_value(a.sx[m]);
        const int64_t idx = (int64_t)m * N + n;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            v[e] = sxm * v[e];
        if (vec) {
            epi_store4(a.ep, a.Y, idx, n, v, false);
        } else {
#pragma unroll 1
            for (int e = 0; e < 4 && n + e < N; ++e)
                epi_store(a.ep, a.Y, idx + e, n + e, v[e]);
        }
    };
    if constexpr (G::KG > 1) {
        float *const red = reinterpret_cast<float *>(ring);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < G::NJ; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    red[kg * G::TM * G::TN +
                        (wm + 32 * i + 8 * (r >> 2) + 4 * hi + (r & 3)) * G::TN + wn + 32 * j +
                        l32] = acc[i][j][r];
        __syncthreads();
#pragma unroll 1
        for (int q = tid; q < G::TM * G::TN / 4; q += G::NT) {
            const f32x4 *const src = reinterpret_cast<const f32x4 *>(red) + q;
            f32x4 v = src[0];
#pragma unroll
            for (int g = 1; g < G::KG; ++g)
                v += src[g * (G::TM * G::TN / 4)];
            store4(m0 + q / (G::TN / 4), n0 + 4 * (q % (G::TN / 4)), v);
        }
    } else {
        float *const patch = reinterpret_cast<float *>(ring) + (tid >> 6) * 1024;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < G::NJ; ++j) {
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    patch[(8 * (r >> 2) + 4 * hi + (r & 3)) * 32 + l32] = acc[i][j][r];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int rl = 8 * t + (lane >> 3);
                    const f32x4 v =
                        *reinterpret_cast<const f32x4 *>(patch + rl * 32 + 4 * (lane & 7));
                    store4(m0 + wm + 32 * i + rl, n0 + wn + 32 * j + 4 * (lane & 7), v);
                }
            }
    }
}

template <class G>
hipError_t launch_pipe(W8Args &b, const W8Plan &p, hipStream_t stream)
{
    b.tiles_m = (int)(((int64_t)b.M + G::TM - 1) / G::TM);
    b.tiles_n = (int)(((int64_t)b.N + G::TN - 1) / G::TN);
    hipLaunchKernelGGL(qgemm_w8a8_pipe_kernel<G>, dim3((unsigned)p.wgs), dim3(G::NT), 0, stream, b);
    return hipGetLastError();
}

// The three shapes of the pipelined kernel (all four wavefronts per SIMD):
//   LARGE  128 x 128 tiles, 8 wavefronts, no K groups, two workgroups per CU:
//          the least operand traffic per output
//   MID    64 x 128 tiles, 4 K groups, one workgroup of 16 wavefronts per CU
//   SMALL  64 x 64 tiles, 8 K groups, likewise
using PipeLarge = PipeGeo<1, 2, 4, 1, 2, 2, 4>;
using PipeMid = PipeGeo<1, 1, 4, 4, 1, 3, 4>;
using PipeSmall = PipeGeo<1, 1, 2, 8, 1, 2, 4>;

// Estimated us of a shape: rounds of one workgroup per CU, each its 64-k
// steps at the measured rate plus a fixed part (prologue, K-group sums,
// store).  Fitted on 16 products (M 64 to 2048, N 512 to 8192, K 512 to 8192);
// measured LARGE / MID / SMALL (before: the general kernel):
//   1290 x 1536 x 1536   19.5 / 12.6 / 15.2 us  (41.0)
//   1290 x 1536 x 6144   58.3 / 35.5 / 43.6     (132)
//   2048 x 8192 x 2048   84.3 / 105  / 126      (116)
//   64 x 4608 x 1536     17.8 / 10.5 / 7.5      (38.7)
template <class G>
void pipe_candidate(const W8Args &a, W8Kernel kernel, double per_step, double fixed, double launch,
                    int cus, W8Plan &best, double &best_us)
{
    const int64_t T = (((int64_t)a.M + G::TM - 1) / G::TM) * (((int64_t)a.N + G::TN - 1) / G::TN);
    const double us =
        (double)((T + cus - 1) / cus) * (a.K / 64 * per_step + fixed) + launch;
    if (T <= W8_MAX_THREADS / G::NT && us < best_us) {
        best = W8Plan{kernel, T, G::NT};
        best_us = us;
    }
}

}  // namespace

// The pipelined kernel in its fastest shape by the estimate, where it takes
// the operands and a shape's launch stays within the threads of a grid (2^30
// rows of one column tile pass it in all three shapes); else the general
// kernel.  A single 64-k step has nothing to pipeline: the general kernel keeps
// up to 8 rows (2 x 1191 x 64 5.0 us, pipelined 5.8) and, where outputs go out
// one at a time (N % 4), grids between one and two of its workgroups per CU
// (1410 x 3915 x 64 18.2 against 20.1; at half the grid 15.5 against 13.7).
W8Plan w8a8_plan(const W8Args &a, int cus)
{
    const int64_t tm = ((int64_t)a.M + BM - 1) / BM, tn = ((int64_t)a.N + BN - 1) / BN;
    W8Plan p{W8_GENERAL, tm * tn, THREADS};
    const bool one_step =
        a.K == 64 && (a.M <= 8 || (a.N % 4 != 0 && p.wgs > cus && p.wgs <= 2 * (int64_t)cus));
    if (a.K % 64 == 0 && a.K < (1 << 23) && ((uintptr_t)a.scales & 3) == 0 && !one_step) {
        double us = 1e300;
        pipe_candidate<PipeLarge>(a, W8_LARGE, 0.62, 0.0, 4.0, cus, p, us);
        pipe_candidate<PipeMid>(a, W8_MID, 0.32, 2.8, 2.0, cus, p, us);
        pipe_candidate<PipeSmall>(a, W8_SMALL, 0.20, 1.9, 2.0, cus, p, us);
    }
    return p;
}

hipError_t launch_qgemm_w8a8(const W8Args &a, int cus, hipStream_t stream)
{
    W8Args b = a;
    const W8Plan p = w8a8_plan(a, cus);
    if (p.wgs <= 0 || p.wgs >= ((int64_t)1 << 31))
        return hipErrorInvalidValue;
    switch (p.kernel) {
    case W8_LARGE: return launch_pipe<PipeLarge>(b, p, stream);
    case W8_MID: return launch_pipe<PipeMid>(b, p, stream);
    case W8_SMALL: return launch_pipe<PipeSmall>(b, p, stream);
    default: break;
    }
    b.tiles_m = (int)(((int64_t)a.M + BM - 1) / BM);
    b.tiles_n = (int)(((int64_t)a.N + BN - 1) / BN);
    hipLaunchKernelGGL(qgemm_w8a8_kernel, dim3((unsigned)p.wgs), dim3(THREADS), 0, stream, b);
    return hipGetLastError();
}

}  // namespace qlk
