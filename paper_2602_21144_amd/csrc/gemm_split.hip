// Float32 products of prefill size on the f16 matrix cores: C = A B^T with every operand value
// written as a sum of two f16 values, three f16 MFMAs in place of the float32 one.
//
// The float32 MFMA runs at 1/16 of the f16 rate, and the float32 tiles of gemm.hip keep it
// 0.91-0.93 busy, so they cannot get faster. Here each operand row is scaled by a power of two
// (its largest magnitude lands in [2^14, 2^15)) and split, x = hi + lo with hi = f16(x) and
// lo = f16(x - hi): 11 + 11 significant bits and the sign of lo, |x - hi - lo| <= 2^-24 |x|
// wherever lo is a normal f16. Then
//     x y = hi_x hi_y + hi_x lo_y + lo_x hi_y   (+ lo_x lo_y <= 2^-24 |x y|, left out),
// all products exact and summed in float32 by v_mfma_f32_16x16x32_f16, and the power of two
// goes back in the epilogue (exact). A sum of K products thus carries about K / 32 x 3 float32
// roundings where the float32 MFMA carries K, and its distance from float64 is smaller:
// measured on N(0, 1) x N(0, 1/K), relative 2-norm, against the float32 tiles: 1.9e-7 and 2.7e-7
// at K = 224, 3.2e-7 and 5.0e-7 at 768, 6.7e-7 and 1.07e-6 at 3584, 1.0e-6 and 1.6e-6 at 8192.
// Times, split and tiles together, against the float32 tiles (0.92 of their peak): 2048x7168x3584
// 770 -> 265 us, 2048x3584x3584 380 -> 148, 512x3584x3584 134 -> 63, 16384x5120x2560 3030 -> 968,
// 1024x3072x768 48 -> 27 us.
//
// Rows the split does not suit (an infinity or NaN, or more than a few nonzero values so far
// below the row's largest that their lo is not a normal f16) are marked in the exponent array;
// the tile kernel leaves their outputs alone and the float32 tiles, launched behind it on the
// same exponents, compute exactly those (and return at once where there are none).
#include <algorithm>

#include "gemm_tiles.h"

namespace ssm {
namespace {

typedef _Float16 f16;
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

constexpr int kSplitBK = 32;  // k per stage: 32 hi and 32 lo halves, one 128-byte line per row

// One workgroup per row of A (rows 0 .. M-1) or B (M .. M+N-1): the row is read once into
// registers (CH pieces of 2048 values), its largest magnitude found, and the halves written as
// [K / 32][hi 32 | lo 32], whole 16-byte pieces. Bound by memory: 4 bytes in, 4 out per value.
template <int CH>
__global__ __launch_bounds__(256) void split_rows_kernel(const float* __restrict__ A, int64_t lda, int M,
                                                         const float* __restrict__ B, int64_t ldb, int K,
                                                         f16* __restrict__ Ap, f16* __restrict__ Bp,
                                                         int32_t* __restrict__ ea, int32_t* __restrict__ eb) {
    __shared__ float smax[4];
    __shared__ int sbad[4];
    const int r = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const bool isa = r < M;
    const int row = isa ? r : r - M;
    const float* src = isa ? A + (int64_t)row * lda : B + (int64_t)row * ldb;
    f16* dst = (isa ? Ap : Bp) + (int64_t)row * 2 * K;
    float v[CH][8];
    float amax = 0.0f;
    bool fin = true;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const int k = (c * 256 + tid) * 8;
        if (k < K) {
            const float4 x = *(const float4*)(src + k), y = *(const float4*)(src + k + 4);
            v[c][0] = x.x; v[c][1] = x.y; v[c][2] = x.z; v[c][3] = x.w;
            v[c][4] = y.x; v[c][5] = y.y; v[c][6] = y.z; v[c][7] = y.w;
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[c][e] = 0.0f;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            amax = fmaxf(amax, fabsf(v[c][e]));
            fin = fin && fabsf(v[c][e]) < __builtin_inff();  // false for NaN too
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off, 64));
    if (lane == 0) smax[wave] = amax;
    const bool wfin = __all(fin);
    __syncthreads();
    amax = fmaxf(fmaxf(smax[0], smax[1]), fmaxf(smax[2], smax[3]));
    // scale 2^-ex puts the largest magnitude into [2^14, 2^15)
    const int ex = amax > 0.0f ? __builtin_amdgcn_frexp_expf(amax) - 15 : 0;
    int small = 0;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const int k = (c * 256 + tid) * 8;
        if (k >= K) continue;
        f16x8 hi, lo;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float x = ldexpf(v[c][e], -ex);
            hi[e] = (f16)x;
            lo[e] = (f16)(x - (float)hi[e]);
            small += x != 0.0f && fabsf(x) < kSplitSmall ? 1 : 0;
        }
        f16* d = dst + (k >> 5) * 64 + (k & 31);
        *(f16x8*)d = hi;
        *(f16x8*)(d + 32) = lo;
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) small += __shfl_xor(small, off, 64);
    if (lane == 0) sbad[wave] = wfin ? small : K + 1;
    __syncthreads();
    if (tid == 0) {
        const int n = sbad[0] + sbad[1] + sbad[2] + sbad[3];
        (isa ? ea : eb)[row] = n > split_small_limit(K) ? kSplitBad : ex;
    }
}

// The tiles: the second schedule of gemm_bf16_dma (every load, fragment read and MFMA in a
// fixed order) over stages of 32 k. A stage's hi and lo fragments are read once each and feed
// three runs of MFMAs: hi x hi while the lo fragments are read; hi x lo, behind the barrier
// (by then every wave has read the whole stage), with the refill of the stage spread between;
// lo x hi, while the next stage's hi fragments are read. The weight fragments' two register
// sets change roles every stage, since the next hi set arrives while this one is in use. Each
// 1 KB moved into LDS serves 1.5 times the MFMAs of a bf16 tile.
template <int ROLE, int BM, int BN, int NS, int WM, int WN>
__global__ __launch_bounds__(64 * WM * WN) void gemm_f16x2_dma(int M, int N, int K, const f16* __restrict__ A,
                                                               const int32_t* __restrict__ ea,
                                                               const f16* __restrict__ B,
                                                               const int32_t* __restrict__ eb, float* __restrict__ C,
                                                               int64_t ldc, int tiles_m, int tiles_n) {
    constexpr int NW = WM * WN, BK = 64;  // halves per LDS row
    constexpr int WTM = BM / WM, WTN = BN / WN, TM = WTM / 16, TN = WTN / 16;
    static_assert(TM * 16 == WTM && TN * 16 == WTN, "whole MFMA blocks per wave");
    constexpr int RPB = 8;  // rows per 1 KB DMA block
    constexpr bool EVEN = BM % (RPB * NW) == 0 && BN % (RPB * NW) == 0;
    constexpr int TBA = BM / RPB, TBT = (BM + BN) / RPB, QM = (TBT + NW - 1) / NW;
    constexpr int AG = EVEN ? BM / RPB / NW : 0, BG = EVEN ? BN / RPB / NW : 0;
    constexpr int OPS = EVEN ? AG + BG : QM;
    static_assert(EVEN || NS == 2, "uneven DMA blocks need the 2-deep ring");
    constexpr int RING = NS * (BM + BN) * BK * 2;
    constexpr int PASSES = (BM * BN * 4 + RING - 1) / RING;
    constexpr int RB = BM / PASSES;
    static_assert(BM % PASSES == 0 && RB % WTM == 0 && (BN * 4) % 128 == 0, "staged output");
    __shared__ __attribute__((aligned(1024))) char smem[RING];
    f16 (*As)[BM * BK] = reinterpret_cast<f16 (*)[BM * BK]>(smem);
    f16 (*Bs)[BN * BK] = reinterpret_cast<f16 (*)[BN * BK]>(smem + NS * BM * BK * 2);

    int tm, tn;
    tile_of(tiles_m, tiles_n, tm, tn);
    const int m0 = tm * BM, n0 = tn * BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WN, wn = wave % WN;
    const int64_t ld = 2 * (int64_t)K;  // halves per packed row
    const int lr = lane >> 3, lp = lane & 7;
    const __amdgpu_buffer_rsrc_t ra = buffer_rsrc(A + (int64_t)m0 * ld, (uint32_t)((int64_t)min(BM, M - m0) * ld * 2));
    const __amdgpu_buffer_rsrc_t rbr = buffer_rsrc(B + (int64_t)n0 * ld, (uint32_t)((int64_t)min(BN, N - n0) * ld * 2));
    // rows past M or N are clamped to a valid row (their results are never stored)
    auto a_off = [&](int r) { return (uint32_t)(((int64_t)(min(m0 + r, M - 1) - m0) * ld + swz_k<BK>(r, lp) * 8) * 2); };
    auto b_off = [&](int r) { return (uint32_t)(((int64_t)(min(n0 + r, N - 1) - n0) * ld + swz_k<BK>(r, lp) * 8) * 2); };
    const uint32_t a_lds = (uint32_t)(uintptr_t)(lds_ptr_t)&As[0][0];
    const uint32_t b_lds = (uint32_t)(uintptr_t)(lds_ptr_t)&Bs[0][0];
    uint32_t aoff[EVEN ? AG : QM], boff[EVEN ? BG : 1];
    const int wu = __builtin_amdgcn_readfirstlane(wave);
    if constexpr (EVEN) {
#pragma unroll
        for (int q = 0; q < AG; ++q) aoff[q] = a_off((wave * AG + q) * RPB + lr);
#pragma unroll
        for (int q = 0; q < BG; ++q) boff[q] = b_off((wave * BG + q) * RPB + lr);
    } else {
#pragma unroll
        for (int q = 0; q < QM; ++q) {
            const int b = wu + NW * q;
            aoff[q] = b < TBA ? a_off(b * RPB + lr) : b_off((b - TBA) * RPB + lr);
        }
    }

    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{};
    const int arow0 = wm * WTM + (lane & 15), brow0 = wn * WTN + (lane & 15);
    const int nk = K / kSplitBK;
    f16x8 fh[TM], fl[TM], fb[2][TN];

    // DMA block d of stage kt into ring slot `slot` (empty resources past the last stage: every
    // wave issues the same number of loads per stage, so every wait is one constant)
    const __amdgpu_buffer_rsrc_t ra_none = buffer_rsrc(A, 0), rb_none = buffer_rsrc(B, 0);
    auto dma_one = [&](int kt, int slot, auto D, __amdgpu_buffer_rsrc_t rA, __amdgpu_buffer_rsrc_t rB)
                       __attribute__((always_inline)) {
        constexpr int d = decltype(D)::value;
        const uint32_t k2 = (uint32_t)(kt * BK) * 2;
        if constexpr (EVEN) {
            if constexpr (d < AG)
                dma16(rA, aoff[d], k2, __builtin_amdgcn_readfirstlane(a_lds + (uint32_t)((slot * BM + (wave * AG + d) * RPB) * BK * 2)));
            else
                dma16(rB, boff[d - AG], k2, __builtin_amdgcn_readfirstlane(b_lds + (uint32_t)((slot * BN + (wave * BG + d - AG) * RPB) * BK * 2)));
        } else {
            const int b = wu + NW * d;
            if (b < TBA)
                dma16(rA, aoff[d], k2, a_lds + (uint32_t)((slot * BM + b * RPB) * BK * 2));
            else if (b < TBT)
                dma16(rB, aoff[d], k2, b_lds + (uint32_t)((slot * BN + (b - TBA) * RPB) * BK * 2));
        }
    };
    auto dma_all = [&](int kt, int slot) __attribute__((always_inline)) {
        const bool live = kt < nk;
        static_for<OPS>([&](auto D) __attribute__((always_inline)) {
            dma_one(kt, slot, D, live ? ra : ra_none, live ? rbr : rb_none);
        });
    };
    // fragment f (activation blocks, then weight blocks) of half h (0 hi, 1 lo) of ring slot
    // `slot`; weight blocks go to register set `set`
    auto frag_one = [&](int slot, auto H, auto SET, auto F) __attribute__((always_inline)) {
        constexpr int h = decltype(H)::value, f = decltype(F)::value;
        const int c = 4 * h + (lane >> 4);
        if constexpr (f < TM) {
            const f16x8 v = *(const f16x8*)&As[slot][(arow0 + f * 16) * BK + swz_k<BK>(arow0, c) * 8];
            if constexpr (h == 0) fh[f] = v;
            else fl[f] = v;
        } else {
            fb[decltype(SET)::value][f - TM] = *(const f16x8*)&Bs[slot][(brow0 + (f - TM) * 16) * BK + swz_k<BK>(brow0, c) * 8];
        }
    };
    constexpr int NMF = TM * TN;
    using Z0 = std::integral_constant<int, 0>;
    using Z1 = std::integral_constant<int, 1>;
    // one run of MFMAs: activation half AH x weight set BSET, with the reads of half RH (weights
    // into RSET) of slot rs (READ) or the refill of slot dst with stage dkt (DMA) in between
    auto run = [&](auto AH, auto BSET, auto READ, auto RH, auto RSET, int rs, auto DMA, int dkt, int dst)
                   __attribute__((always_inline)) {
        const bool live = dkt < nk;
        const __amdgpu_buffer_rsrc_t rA = live ? ra : ra_none, rB = live ? rbr : rb_none;
        static_for<NMF>([&](auto Q) __attribute__((always_inline)) {
            constexpr int q = decltype(Q)::value, i = q / TN, j = q % TN;
            if constexpr (decltype(DMA)::value)
                static_for<OPS>([&](auto D) __attribute__((always_inline)) {
                    if constexpr (decltype(D)::value * NMF / OPS == q) dma_one(dkt, dst, D, rA, rB);
                });
            if constexpr (decltype(READ)::value)
                static_for<TM + TN>([&](auto F) __attribute__((always_inline)) {
                    if constexpr ((decltype(F)::value < NMF ? decltype(F)::value : NMF - 1) == q) frag_one(rs, RH, RSET, F);
                });
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fb[decltype(BSET)::value][j],
                                                               decltype(AH)::value ? fl[i] : fh[i], acc[i][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    // stage kt in ring slot cur; its hi fragments are in fh and fb[P] on entry, the next stage's
    // in fh and fb[1 - P] on exit
    auto stage = [&](int kt, auto P) __attribute__((always_inline)) {
        constexpr int p = decltype(P)::value;
        using SP = std::integral_constant<int, p>;
        using SQ = std::integral_constant<int, 1 - p>;
        const int cur = kt % NS;
        run(Z0{}, SP{}, std::true_type{}, Z1{}, SQ{}, cur, std::false_type{}, 0, 0);
        // stage kt+1 has landed (this wave's loads, then all waves') and every wave has read
        // stage kt, so its slot can be refilled
        wait_vm<(NS - 2) * OPS>();
        wait_lgkm0();
        __syncthreads();
        run(Z0{}, SQ{}, std::false_type{}, Z0{}, SP{}, 0, std::true_type{}, kt + NS, cur);
        run(Z1{}, SP{}, std::true_type{}, Z0{}, SQ{}, (kt + 1) % NS, std::false_type{}, 0, 0);
    };
    static_for<NS - 1>([&](auto ST) __attribute__((always_inline)) { dma_all(ST, ST); });
    wait_vm<(NS - 2) * OPS>();  // stage 0 complete
    dma_all(NS - 1, NS - 1);
    __syncthreads();
    static_for<TM + TN>([&](auto F) __attribute__((always_inline)) { frag_one(0, Z0{}, Z0{}, F); });
    int kt = 0;
    for (; kt + 1 < nk; kt += 2) {
        stage(kt, Z0{});
        stage(kt + 1, Z1{});
    }
    if (kt < nk) stage(kt, Z0{});
    wait_vm<0>();  // the loads of nothing past the last stage write the ring too

    // The output tile goes through LDS in whole-line pieces (row r as 16-byte chunks, chunk c at
    // c ^ (r & 7)); the rows' and columns' powers of two go in on the way.
    float* st = reinterpret_cast<float*>(smem);
    constexpr int CPR_O = BN / 4;
    const bool vec = ((uintptr_t)C & 15) == 0 && ldc % 4 == 0;
    bool bad = false;
    int en[TN][4];
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int n = n0 + wn * WTN + j * 16 + 4 * (lane >> 4) + e;
            en[j][e] = n < N ? eb[n] : 0;
            bad = bad || en[j][e] == kSplitBad;
        }
#pragma unroll
    for (int pass = 0; pass < PASSES; ++pass) {
        __syncthreads();  // every wave is done with the ring (then with the previous pass)
        if (wm * WTM >= pass * RB && wm * WTM < (pass + 1) * RB) {
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int r = wm * WTM - pass * RB + i * 16 + (lane & 15);
                const int m = m0 + pass * RB + r;
                const int em = m < M ? ea[m] : 0;
                bad = bad || em == kSplitBad;
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const int col = wn * WTN + j * 16 + 4 * (lane >> 4);
                    *(float4*)(st + r * BN + (((col / 4) ^ (r & 7)) * 4)) =
                        make_float4(ldexpf(acc[i][j][0], em + en[j][0]), ldexpf(acc[i][j][1], em + en[j][1]),
                                    ldexpf(acc[i][j][2], em + en[j][2]), ldexpf(acc[i][j][3], em + en[j][3]));
                }
            }
        }
        const bool any_bad = __syncthreads_or(bad);
        for (int c = tid; c < RB * CPR_O; c += 64 * NW) {
            const int r = c / CPR_O, cc = c % CPR_O;
            const int m = m0 + pass * RB + r, n = n0 + cc * 4;
            if (m >= M || n >= N) continue;
            const float* q = st + r * BN + ((cc ^ (r & 7)) * 4);
            float* p = C + (int64_t)m * ldc + n;
            if (vec && n + 4 <= N && !any_bad) {
                *(float4*)p = *(const float4*)q;
            } else {
                // outputs of marked rows and columns are the float32 tiles'
                const bool row_ok = ea[m] != kSplitBad;
                for (int e = 0; e < 4 && n + e < N; ++e)
                    if (row_ok && eb[n + e] != kSplitBad) p[e] = q[e];
            }
        }
    }
}

// The tiles, priced as those of the bf16 table (gemm.hip) by times fitted over 140 shapes,
// M = 130 .. 16384, N = 256 .. 16384, K = 224 .. 8192; a per 32-wide stage. The cheapest is
// within 1% of the best on average (9% at worst). 256x256 reaches 8.9 TFLOP/s of f16 products
// per CU (2.3 PFLOP/s over the card; a bf16 tile, which moves 1.5 times the bytes per product,
// 6.3), 64x64 3.3.
enum SplitTile { kS64x64, kS64x128, kS96x128, kS128x128, kS192x128, kS256x128, kS192x256, kS256x256, kSplitTiles };
struct SplitCost {
    int bm, bn;
    float a, a2, b;  // a2: per stage when two tiles share a CU (0: the ring fills it)
};
constexpr SplitCost kSplitCost[kSplitTiles] = {
    {64, 64, 0.239f, 0.383f, 1.54f},  {64, 128, 0.347f, 0.0f, 3.03f},  {96, 128, 0.473f, 0.0f, 4.66f},
    {128, 128, 0.553f, 0.0f, 4.31f},  {192, 128, 0.738f, 0.0f, 5.37f}, {256, 128, 0.860f, 0.0f, 7.02f},
    {192, 256, 1.105f, 0.0f, 9.65f},  {256, 256, 1.421f, 0.0f, 11.77f}};

float split_tile_us(const SplitCost& t, int64_t M, int64_t N, int64_t K) {
    const int64_t wg = ((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn);
    const float nk = (float)(K / kSplitBK);
    const float r = wg <= 4 * 256 ? (float)((wg + 255) / 256) : (float)wg / 256.0f + 0.6f;
    if (t.a2 > 0.0f && wg > 256) {
        const float pairs = wg < 2048 ? (float)((wg + 511) / 512) : (float)wg / 512.0f + 0.5f;
        return 2.0f + pairs * t.a2 * nk + r * t.b;
    }
    return 2.0f + r * (t.a * nk + t.b);
}

SplitTile pick_split_tile(int64_t M, int64_t N, int64_t K, float* us) {
    int best = 0;
    float bu = 1e30f;
    for (int i = 0; i < kSplitTiles; ++i) {
        const float u = split_tile_us(kSplitCost[i], M, N, K);
        if (u < bu) { bu = u; best = i; }
    }
    *us = bu;
    return (SplitTile)best;
}

template <int ROLE, int BM, int BN, int NS, int WM, int WN>
hipError_t run_split(int64_t M, int64_t N, int64_t K, const SplitOperands& o, float* C, int64_t ldc, hipStream_t s) {
    const int tm = (int)((M + BM - 1) / BM), tn = (int)((N + BN - 1) / BN);
    SSM_LAUNCH((gemm_f16x2_dma<ROLE, BM, BN, NS, WM, WN>), dim3(tm * tn), dim3(64 * WM * WN), 0, s, (int)M, (int)N,
               (int)K, (const f16*)o.a, o.ea, (const f16*)o.b, o.eb, C, ldc, tm, tn);
    return hipGetLastError();
}

template <int ROLE>
hipError_t dispatch_split(SplitTile t, int64_t M, int64_t N, int64_t K, const SplitOperands& o, float* C, int64_t ldc,
                          hipStream_t s) {
    switch (t) {
        case kS64x64: return run_split<ROLE, 64, 64, 4, 2, 2>(M, N, K, o, C, ldc, s);
        case kS64x128: return run_split<ROLE, 64, 128, 4, 2, 4>(M, N, K, o, C, ldc, s);
        case kS96x128: return run_split<ROLE, 96, 128, 4, 2, 2>(M, N, K, o, C, ldc, s);
        case kS128x128: return run_split<ROLE, 128, 128, 3, 2, 4>(M, N, K, o, C, ldc, s);
        case kS192x128: return run_split<ROLE, 192, 128, 3, 2, 4>(M, N, K, o, C, ldc, s);
        case kS256x128: return run_split<ROLE, 256, 128, 2, 4, 2>(M, N, K, o, C, ldc, s);
        case kS192x256: return run_split<ROLE, 192, 256, 2, 2, 4>(M, N, K, o, C, ldc, s);
        default: return run_split<ROLE, 256, 256, 2, 2, 4>(M, N, K, o, C, ldc, s);
    }
}

}  // namespace

size_t gemm_f32_halves_bytes(int64_t M, int64_t N, int64_t K) {
    if (M <= 64 || K % kSplitBK != 0 || K > kSplitMaxK) return 0;
    return (size_t)(M + N) * K * 4 + align256((size_t)M * 4) + align256((size_t)N * 4);
}

float gemm_f32_split_us(int64_t M, int64_t N, int64_t K) {
    float us;
    pick_split_tile(M, N, K, &us);
    // the rows' split at 6.2 TB/s (4 bytes in, 4 out per value) and its launch, the tiles, and
    // the float32 tiles' launch that finds nothing to do
    return us + 2.0f + (float)((M + N) * K) * (8.0f / 6.2e6f) + 2.5f;
}

hipError_t launch_gemm_f32_split(int role, int64_t M, int64_t N, int64_t K, const float* A, int64_t lda, const float* B,
                                 int64_t ldb, float* C, int64_t ldc, void* halves, hipStream_t s, SplitOperands* out) {
    char* b = (char*)halves;
    SplitOperands o;
    o.a = b; b += (size_t)M * K * 4;
    o.b = b; b += (size_t)N * K * 4;
    o.ea = (int32_t*)b; b += align256((size_t)M * 4);
    o.eb = (int32_t*)b;
    *out = o;
    {
        KernelTimer kt("gemm.split_rows", s);
        const dim3 grid((unsigned)(M + N)), block(256);
#define SSM_SPLIT_ROWS(CH) \
    SSM_LAUNCH(split_rows_kernel<CH>, grid, block, 0, s, A, lda, (int)M, B, ldb, (int)K, (f16*)o.a, (f16*)o.b, o.ea, o.eb)
        if (K <= 2048) SSM_SPLIT_ROWS(1);
        else if (K <= 4096) SSM_SPLIT_ROWS(2);
        else SSM_SPLIT_ROWS(4);
#undef SSM_SPLIT_ROWS
        if (const hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    }
    float us;
    const SplitTile t = pick_split_tile(M, N, K, &us);
    switch (role) {
        case kGemmXProj: return dispatch_split<kGemmXProj>(t, M, N, K, o, C, ldc, s);
        case kGemmDtProj: return dispatch_split<kGemmDtProj>(t, M, N, K, o, C, ldc, s);
        case kGemmOutProj: return dispatch_split<kGemmOutProj>(t, M, N, K, o, C, ldc, s);
        default: return dispatch_split<kGemmInProj>(t, M, N, K, o, C, ldc, s);
    }
}

}  // namespace ssm
