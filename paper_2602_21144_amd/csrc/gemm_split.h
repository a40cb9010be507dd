// Float32 products of prefill size on the bf16 matrix cores: C = A B^T with every operand value
// written as the sum of three bf16 values, six bf16 MFMAs in place of the float32 ones.
//
// The float32 MFMA runs at 1/16 of the bf16 rate, and the float32 tiles of gemm.hip keep it
// 0.91-0.93 busy, so they cannot get faster. Here x = x1 + x2 + x3 with x1 = bf16(x),
// x2 = bf16(x - x1), x3 = bf16(x - x1 - x2), round to nearest: 8 + 8 + 8 significant bits hold all
// 24 of a float32, whatever the other values of its row, because bf16 has float32's exponents. (Two
// f16 values hold 22 bits, and fewer for a value far below the largest of its row.) Then
//     x y = x1 y1 + (x1 y2 + x2 y1) + (x2 y2 + x1 y3 + x3 y1)   (+ x2 y3 + x3 y2 + x3 y3),
// where |x2| <= 2^-9 |x| and |x3| <= 2^-18 |x|, so that what is left out is below 2^-25.9 |x y|, a
// quarter of the rounding of one float32 product. All products are exact and summed in float32 by
// v_mfma_f32_16x16x32_bf16, 6 roundings of a sum per 32 products.
//
// The values are split behind the fragment reads, so operands move as the float32 rows they are:
// no pass over them, no copy of them in memory. x is first scaled by 2^24 (exact), which keeps x3
// a normal bf16 down to the smallest float32; the sums carry 2^48, taken out in the epilogue.
// Values from 2^104 on, infinities, NaN, and sums from 2^80 on give an infinity or NaN, and nothing
// else does: a tile with one is computed again on the float32 MFMA by the same workgroup
// (2048x7168x3584: 451-490 us, 1190 with one such row, or with all; the float32 tiles alone 805-820).
//
// Distance from float64 (relative 2-norm, N(0, 1) x N(0, 1/K)) against the float32 tiles: 2.1e-7 and
// 2.7e-7 at K = 224, 9.4e-7 and 1.07e-6 at 3584. Times against them: 2048x7168x3584 805 -> 451 us,
// 2048x3584x3584 363 -> 264 (two K-slices), 16384x2560x2560 1518 -> 934, 391x10240x2560 260 -> 143,
// 2048x3584x224 32 -> 27.
#pragma once
#include "gemm_tiles.h"

namespace ssm {
namespace {

constexpr float kSplitScale = 0x1p24f, kSplitUnscale = 0x1p-48f;

// Two values rounded to bf16. The empty assembly hides where the bits come from: the compiler would
// round one of the values a second time where it is taken back to float32.
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    typedef bf16 bf16x2 __attribute__((ext_vector_type(2)));
    bf16x2 v;
    v[0] = (bf16)a; v[1] = (bf16)b;
    uint32_t o = __builtin_bit_cast(uint32_t, v);
    asm("" : "+v"(o));
    return o;
}
__device__ __forceinline__ float bits_f32(uint32_t b) { return __builtin_bit_cast(float, b); }

// The tiles: 256 rows of A by BN rows of B, four waves of 128 x BN/2, one per SIMD, over a 2-deep
// ring of stages on the DMA path (as in gemm_bf16_dma), with every load, fragment read, piece of a
// split and MFMA in a fixed order. The split is 6.5 VALU instructions per value, 52 per fragment
// of a lane, and every wave splits its own fragments, so wide wave tiles are what keeps the matrix
// cores ahead of it: at BN = 224, 8 + 7 fragments are 3120 VALU cycles (and 1340 of MFMA issue)
// beside the 5380 MFMA cycles of 56 blocks; eight waves of 128x64 (256x256) have 2500 + 770 beside
// 3070 and took 521 us for 2048x7168x3584 where this form takes 451. That is 1.4 PFLOP/s of bf16
// products, the rate that these tiles reach on bf16 operands too.
// A stage is a sequence of TN + 8 splits, each spread over the MFMAs of one slot, its fragment read
// one slot ahead: block rows 0 to 3 column by column while the weight fragments 1 .. TN-1 and row 4
// are split, then rows 4 to 7, two splits in each: rows 5, 6, 7, of the next stage rows 2, 3, 0, 1 and
// weight fragment 0. Between rows 4 and 5 every wave has read the stage, and its slot is refilled.
// Workgroup (tile, blockIdx.y) takes K-slice blockIdx.y (K is its length) into its own C.
template <int ROLE, int BN>
__global__ __launch_bounds__(256, 1) void gemm_f32x3_dma(int M, int N, int K, const float* __restrict__ A, int64_t lda,
                                                         const float* __restrict__ B, int64_t ldb,
                                                         float* __restrict__ C, int64_t ldc, int tiles_m, int tiles_n) {
    constexpr int BM = 256, WM = 2, WN = 2, NS = 2;
    constexpr int NW = WM * WN, BK = 64;  // 2-byte units per LDS row
    constexpr int WTM = BM / WM, WTN = BN / WN, TM = WTM / 16, TN = WTN / 16;
    static_assert(TM * 16 == WTM && TN * 16 == WTN && TM == 8 && TN >= 4, "eight block rows per wave");
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
    char* const As = smem;
    char* const Bs = smem + NS * BM * BK * 2;

    A += (int64_t)blockIdx.y * K;
    B += (int64_t)blockIdx.y * K;
    C += (int64_t)blockIdx.y * M * ldc;
    int tm, tn;
    tile_of(tiles_m, tiles_n, tm, tn);
    const int m0 = tm * BM, n0 = tn * BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WN, wn = wave % WN;
    const int lr = lane >> 3, lp = lane & 7;
    const __amdgpu_buffer_rsrc_t ra = buffer_rsrc(A + (int64_t)m0 * lda, (uint32_t)((int64_t)min(BM, M - m0) * lda * 4));
    const __amdgpu_buffer_rsrc_t rbr = buffer_rsrc(B + (int64_t)n0 * ldb, (uint32_t)((int64_t)min(BN, N - n0) * ldb * 4));
    // rows past M or N are clamped to a valid row (their results are never stored)
    auto a_off = [&](int r) { return (uint32_t)((min(m0 + r, M - 1) - m0) * lda * 4 + swz_k<BK>(r, lp) * 16); };
    auto b_off = [&](int r) { return (uint32_t)((min(n0 + r, N - 1) - n0) * ldb * 4 + swz_k<BK>(r, lp) * 16); };
    const uint32_t a_lds = (uint32_t)(uintptr_t)(lds_ptr_t)As;
    const uint32_t b_lds = (uint32_t)(uintptr_t)(lds_ptr_t)Bs;
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
    const int arow0 = wm * WTM + (lane & 15), brow0 = wn * WTN + (lane & 15);
    const int nk = K / kSplitBK;

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
    // A lane's 8 values of block i: chunks g and g + 4 of its row, g = lane / 16. Both operands take
    // the same ones, so which k a value stands for does not matter.
    struct Raw { f32x4 v[2]; };
    struct Parts { u32x4 t[3]; };
    const int sw0 = swz_k<BK>(lane & 15, lane >> 4) * 16, sw1 = swz_k<BK>(lane & 15, 4 + (lane >> 4)) * 16;
    auto read_a = [&](Raw& r, int slot, int i) __attribute__((always_inline)) {
        const char* p = As + (slot * BM + arow0 + i * 16) * BK * 2;
        r.v[0] = *(const f32x4*)(p + sw0);
        r.v[1] = *(const f32x4*)(p + sw1);
    };
    auto read_b = [&](Raw& r, int slot, int j) __attribute__((always_inline)) {
        const char* p = Bs + (slot * BN + brow0 + j * 16) * BK * 2;
        r.v[0] = *(const f32x4*)(p + sw0);
        r.v[1] = *(const f32x4*)(p + sw1);
    };
    // piece it of 12 of a split: part it / 4 of pair it % 4 (r holds what is left of the values)
    constexpr int kPieces = 12;
    auto piece = [&](auto IT, Raw& r, Parts& o) __attribute__((always_inline)) {
        constexpr int part = decltype(IT)::value / 4, p = decltype(IT)::value % 4;
        float& x = reinterpret_cast<float(&)[8]>(r)[2 * p];
        float& y = reinterpret_cast<float(&)[8]>(r)[2 * p + 1];
        if constexpr (part == 0) {
            x *= kSplitScale;
            y *= kSplitScale;
        } else {
            const uint32_t t = o.t[part - 1][p];
            x -= bits_f32(t << 16);
            y -= bits_f32(t & 0xffff0000u);
        }
        o.t[part][p] = pack_bf16(x, y);
    };
    auto mma = [&](auto T, int i, int j, const Parts& a, const Parts& b) __attribute__((always_inline)) {
        // the small products first
        constexpr int ta[6] = {2, 0, 1, 1, 0, 0}, tb[6] = {0, 2, 1, 0, 1, 0};
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, b.t[tb[decltype(T)::value]]),
                                                            __builtin_bit_cast(bf16x8, a.t[ta[decltype(T)::value]]),
                                                            acc[i][j], 0, 0, 0);
    };
    Raw x[2];
    Parts fa[5], fb[TN];
    // split s of a stage (1 .. TN + 8) and its fragment: x[(s + P) & 1], P the stage's parity
    auto read_item = [&](auto S, auto P, int cur, int nxt) __attribute__((always_inline)) {
        constexpr int s = decltype(S)::value;
        constexpr int row[8] = {4, 5, 6, 7, 2, 3, 0, 1};
        Raw& r = x[(s + decltype(P)::value) & 1];
        if constexpr (s < TN) read_b(r, cur, s);
        else if constexpr (s < TN + 8) read_a(r, s < TN + 4 ? cur : nxt, row[s - TN]);
        else read_b(r, nxt, s - TN - 8);
    };
    auto split_piece = [&](auto S, auto P, auto IT) __attribute__((always_inline)) {
        constexpr int s = decltype(S)::value;
        constexpr int set[8] = {4, 0, 1, 4, 2, 3, 0, 1};
        Raw& r = x[(s + decltype(P)::value) & 1];
        if constexpr (s < TN) piece(IT, r, fb[s]);
        else if constexpr (s < TN + 8) piece(IT, r, fa[set[s - TN]]);
        else piece(IT, r, fb[0]);
    };
    // MFMA q of n of slot S: the pieces of its split, then the MFMA
    auto pieces_at = [&](auto S, auto P, auto Q, auto N_) __attribute__((always_inline)) {
        static_for<kPieces>([&](auto IT) __attribute__((always_inline)) {
            if constexpr (decltype(IT)::value * decltype(N_)::value / kPieces == decltype(Q)::value) split_piece(S, P, IT);
        });
    };
    constexpr int NMF = 6 * TN, H0 = NMF / 2;  // MFMAs of a block row, of its first slot
    auto stage = [&](int kt, auto P) __attribute__((always_inline)) {
        const int cur = kt % NS, nxt = (kt + 1) % NS;
        static_for<TN>([&](auto J) __attribute__((always_inline)) {
            constexpr int j = decltype(J)::value;
            read_item(std::integral_constant<int, j + 2>{}, P, cur, nxt);
            static_for<24>([&](auto Q) __attribute__((always_inline)) {
                constexpr int q = decltype(Q)::value;
                pieces_at(std::integral_constant<int, j + 1>{}, P, Q, std::integral_constant<int, 24>{});
                mma(std::integral_constant<int, q / 4>{}, q % 4, j, fa[q % 4], fb[j]);
                __builtin_amdgcn_sched_barrier(0);
            });
        });
        const bool live = kt + NS < nk;
        const __amdgpu_buffer_rsrc_t rA = live ? ra : ra_none, rB = live ? rbr : rb_none;
        static_for<4>([&](auto I) __attribute__((always_inline)) {
            constexpr int i = 4 + decltype(I)::value, s = TN + 1 + 2 * (i - 4);
            constexpr int set[4] = {4, 0, 1, 4};
            if constexpr (i == 5) {
                // stage kt+1 has landed (this wave's loads, then all waves') and every wave has read
                // stage kt, so its slot can be refilled
                wait_vm<(NS - 2) * OPS>();
                wait_lgkm0();
                __syncthreads();
            }
            static_for<NMF>([&](auto Q) __attribute__((always_inline)) {
                constexpr int q = decltype(Q)::value;
                using S0 = std::integral_constant<int, s>;
                using S1 = std::integral_constant<int, s + 1>;
                if constexpr (q == 0) read_item(S1{}, P, cur, nxt);
                if constexpr (q == H0) read_item(std::integral_constant<int, s + 2>{}, P, cur, nxt);
                if constexpr (i >= 5)
                    static_for<OPS>([&](auto D) __attribute__((always_inline)) {
                        if constexpr (decltype(D)::value * 3 * NMF / OPS == (i - 5) * NMF + q) dma_one(kt + NS, cur, D, rA, rB);
                    });
                if constexpr (q < H0) pieces_at(S0{}, P, Q, std::integral_constant<int, H0>{});
                else pieces_at(S1{}, P, std::integral_constant<int, q - H0>{}, std::integral_constant<int, NMF - H0>{});
                // the last row column by column, so that weight fragment 0 is free for the next stage's
                if constexpr (i < 7) mma(std::integral_constant<int, q / TN>{}, i, q % TN, fa[set[i - 4]], fb[q % TN]);
                else {
                    constexpr int c = q / 12 * 2;
                    constexpr bool two = c + 1 < TN;
                    mma(std::integral_constant<int, two ? (q % 12) / 2 : q % 12>{}, i, two ? c + q % 2 : c, fa[4], fb[two ? c + q % 2 : c]);
                }
                __builtin_amdgcn_sched_barrier(0);
            });
        });
    };
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{};
    static_for<NS - 1>([&](auto ST) __attribute__((always_inline)) { dma_all(ST, ST); });
    wait_vm<(NS - 2) * OPS>();  // stage 0 complete
    dma_all(NS - 1, NS - 1);
    __syncthreads();
    using Z0 = std::integral_constant<int, 0>;
    using Z1 = std::integral_constant<int, (TN + 8) % 2>;  // an odd number of splits flips x
    static_for<5>([&](auto I) __attribute__((always_inline)) {
        constexpr int i = decltype(I)::value;
        if constexpr (i < 4) read_a(x[0], 0, i);
        else read_b(x[0], 0, 0);
        static_for<kPieces>([&](auto IT) __attribute__((always_inline)) { piece(IT, x[0], i < 4 ? fa[i] : fb[0]); });
    });
    read_item(std::integral_constant<int, 1>{}, Z0{}, 0, 0);
    int kt = 0;
    for (; kt + 1 < nk; kt += 2) {
        stage(kt, Z0{});
        stage(kt + 1, Z1{});
    }
    if (kt < nk) stage(kt, Z0{});
    wait_vm<0>();  // the loads of nothing past the last stage write the ring too

    // The output tile goes through LDS in whole-line pieces (row r as 16-byte chunks, chunk c at
    // c ^ (r & 7)).
    auto store = [&](const f32x4 (&o)[TM][TN], float scale) __attribute__((always_inline)) {
        float* st = reinterpret_cast<float*>(smem);
        constexpr int CPR_O = BN / 4;
        const bool vec = ((uintptr_t)C & 15) == 0 && ldc % 4 == 0;
#pragma unroll
        for (int pass = 0; pass < PASSES; ++pass) {
            __syncthreads();  // every wave is done with the ring (then with the previous pass)
            if (wm * WTM >= pass * RB && wm * WTM < (pass + 1) * RB) {
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    const int r = wm * WTM - pass * RB + i * 16 + (lane & 15);
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        const int col = wn * WTN + j * 16 + 4 * (lane >> 4);
                        *(float4*)(st + r * BN + (((col / 4) ^ (r & 7)) * 4)) =
                            make_float4(o[i][j][0] * scale, o[i][j][1] * scale, o[i][j][2] * scale, o[i][j][3] * scale);
                    }
                }
            }
            __syncthreads();
            for (int c = tid; c < RB * CPR_O; c += 64 * NW) {
                const int r = c / CPR_O, cc = c % CPR_O;
                const int m = m0 + pass * RB + r, n = n0 + cc * 4;
                if (m >= M || n >= N) continue;
                const float* q = st + r * BN + ((cc ^ (r & 7)) * 4);
                float* p = C + (int64_t)m * ldc + n;
                if (vec && n + 4 <= N) {
                    *(float4*)p = *(const float4*)q;
                } else {
                    for (int e = 0; e < 4 && n + e < N; ++e) p[e] = q[e];
                }
            }
        }
    };
    // an infinity or NaN among the sums: the tile again, on float32
    float z = 0.0f;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) z = __builtin_fmaf(acc[i][j][e], 0.0f, z);
    if (!__syncthreads_or(!(z == 0.0f))) {
        store(acc, kSplitUnscale);
        return;
    }
    f32x4 sum[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) sum[i][j] = f32x4{};
    static_for<NS - 1>([&](auto ST) __attribute__((always_inline)) { dma_all(ST, ST); });
    for (int kt = 0; kt < nk; ++kt) {
        wait_vm<(NS - 2) * OPS>();
        wait_lgkm0();
        __syncthreads();  // stage kt has landed, and stage kt - 1 is read
        dma_all(kt + NS - 1, (kt + NS - 1) % NS);
        Raw b[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) read_b(b[j], kt % NS, j);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            Raw a;
            read_a(a, kt % NS, i);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int e = 0; e < 8; ++e)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    sum[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[j].v[e / 4][e % 4], a.v[e / 4][e % 4],
                                                                     sum[i][j], 0, 0, 0);
        }
    }
    wait_vm<0>();
    store(sum, 1.0f);
}

template <int ROLE, int BN>
hipError_t run_parts(int slices, int64_t M, int64_t N, int64_t K, const float* A, int64_t lda, const float* B,
                     int64_t ldb, float* C, int64_t ldc, hipStream_t s) {
    const int tm = (int)((M + 255) / 256), tn = (int)((N + BN - 1) / BN);
    SSM_LAUNCH((gemm_f32x3_dma<ROLE, BN>), dim3(tm * tn, slices), dim3(256), 0, s, (int)M, (int)N, (int)(K / slices), A,
               lda, B, ldb, C, ldc, tm, tn);
    return hipGetLastError();
}

}  // namespace

// The product on tiles of one width. Each width is instantiated in a file of its own (gemm_split_*.hip): a
// tile is 7 to 21 s of compiling, and the 16 of them in one file took eight minutes.
template <int BN>
hipError_t launch_parts_tile(int role, int slices, int64_t M, int64_t N, int64_t K, const float* A, int64_t lda,
                             const float* B, int64_t ldb, float* C, int64_t ldc, hipStream_t s) {
    switch (role) {
        case kGemmXProj: return run_parts<kGemmXProj, BN>(slices, M, N, K, A, lda, B, ldb, C, ldc, s);
        case kGemmDtProj: return run_parts<kGemmDtProj, BN>(slices, M, N, K, A, lda, B, ldb, C, ldc, s);
        case kGemmOutProj: return run_parts<kGemmOutProj, BN>(slices, M, N, K, A, lda, B, ldb, C, ldc, s);
        default: return run_parts<kGemmInProj, BN>(slices, M, N, K, A, lda, B, ldb, C, ldc, s);
    }
}

}  // namespace ssm
