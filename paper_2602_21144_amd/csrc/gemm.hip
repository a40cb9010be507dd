// Dense projections of the mixer (in_proj, x_proj, dt_proj, out_proj) as
// C[M][N] = A[M][K] * B[N][K]^T on gfx950 matrix cores.
//
// Both operands are K-contiguous (activations [tokens][features], weights
// [out_features][in_features]), which is the natural operand layout of MFMA: every
// lane loads 8 consecutive k of one row. bf16 path: v_mfma_f32_32x32x16_bf16 with
// fp32 accumulation; fp32 path: v_mfma_f32_16x16x4_f32.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "gemm_tiles.h"

namespace ssm {
namespace {

constexpr int kBK = 64;  // k per LDS stage (bf16): 128 bytes per row = 8 chunks of 16 B

// Row r of an LDS tile stores its 8 chunks permuted by an XOR with (r>>1)&7, so the
// 16 lanes that read one chunk column from 16 consecutive rows hit distinct banks.
__device__ __forceinline__ int swz(int row, int chunk) { return chunk ^ ((row >> 1) & 7); }

__device__ __forceinline__ bf16x8 cvt8(float4 a, float4 b) {
    bf16x8 o;
    o[0] = (bf16)a.x; o[1] = (bf16)a.y; o[2] = (bf16)a.z; o[3] = (bf16)a.w;
    o[4] = (bf16)b.x; o[5] = (bf16)b.y; o[6] = (bf16)b.z; o[7] = (bf16)b.w;
    return o;
}

// ROLE only names the instance (one kernel symbol per projection, so profiles separate them).
template <int ROLE, int BM, int BN, int WM, int WN, bool A_F32, bool C_F32>
__global__ __launch_bounds__(256) void gemm_bf16_nt(int M, int N, int K,
                                                    const void* __restrict__ Ap, int64_t lda,
                                                    const bf16* __restrict__ B, int64_t ldb,
                                                    void* __restrict__ Cp, int64_t ldc,
                                                    int tiles_m, int tiles_n) {
    static_assert(WM * WN == 4, "four waves");
    constexpr int WTM = BM / WM, WTN = BN / WN;
    constexpr int TM = WTM / 32, TN = WTN / 32;
    static_assert(TM >= 1 && TN >= 1 && WTM % 32 == 0 && WTN % 32 == 0, "wave tile");
    constexpr int AC = BM * 8 / 256;  // 16-byte chunks per thread per stage
    constexpr int BC = BN * 8 / 256;
    static_assert(AC >= 1 && BC >= 1, "tile too small for 256 threads");

    __shared__ __attribute__((aligned(16))) bf16 As[2][BM * kBK];
    __shared__ __attribute__((aligned(16))) bf16 Bs[2][BN * kBK];

    int tm, tn;
    tile_of(tiles_m, tiles_n, tm, tn);
    const int m0 = tm * BM, n0 = tn * BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WN, wn = wave % WN;

    bf16x8 ra[AC], rb[BC];

    auto gload = [&](int k0) {
#pragma unroll
        for (int i = 0; i < AC; ++i) {
            const int q = tid + 256 * i, row = q >> 3, ck = q & 7;
            const int gm = m0 + row, gk = k0 + ck * 8;
            if (gm < M && gk < K) {
                if constexpr (A_F32) {
                    const float* p = (const float*)Ap + (int64_t)gm * lda + gk;
                    ra[i] = cvt8(*(const float4*)p, *(const float4*)(p + 4));
                } else {
                    ra[i] = *(const bf16x8*)((const bf16*)Ap + (int64_t)gm * lda + gk);
                }
            } else {
                ra[i] = bf16x8{};
            }
        }
#pragma unroll
        for (int i = 0; i < BC; ++i) {
            const int q = tid + 256 * i, row = q >> 3, ck = q & 7;
            const int gn = n0 + row, gk = k0 + ck * 8;
            rb[i] = (gn < N && gk < K) ? *(const bf16x8*)(B + (int64_t)gn * ldb + gk) : bf16x8{};
        }
    };
    auto lstore = [&](int buf) {
#pragma unroll
        for (int i = 0; i < AC; ++i) {
            const int q = tid + 256 * i, row = q >> 3, ck = q & 7;
            *(bf16x8*)&As[buf][row * kBK + swz(row, ck) * 8] = ra[i];
        }
#pragma unroll
        for (int i = 0; i < BC; ++i) {
            const int q = tid + 256 * i, row = q >> 3, ck = q & 7;
            *(bf16x8*)&Bs[buf][row * kBK + swz(row, ck) * 8] = rb[i];
        }
    };

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x16{};

    const int nk = (K + kBK - 1) / kBK;
    gload(0);
    lstore(0);
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
        const int cur = kt & 1;
        if (kt + 1 < nk) gload((kt + 1) * kBK);
#pragma unroll
        for (int s = 0; s < kBK / 16; ++s) {
            const int c = s * 2 + (lane >> 5);
            bf16x8 af[TM], bfg[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int row = wm * WTM + i * 32 + (lane & 31);
                af[i] = *(const bf16x8*)&As[cur][row * kBK + swz(row, c) * 8];
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int row = wn * WTN + j * 32 + (lane & 31);
                bfg[j] = *(const bf16x8*)&Bs[cur][row * kBK + swz(row, c) * 8];
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfg[j], af[i], acc[i][j], 0, 0, 0);
        }
        if (kt + 1 < nk) lstore(cur ^ 1);
        __syncthreads();
    }

    // Operands were swapped (B rows first), so lane l holds output row (l & 31) and
    // four consecutive output columns per group of four accumulators.
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int m = m0 + wm * WTM + i * 32 + (lane & 31);
        if (m >= M) continue;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int n = n0 + wn * WTN + j * 32 + 8 * g + 4 * (lane >> 5);
                const float v0 = acc[i][j][4 * g], v1 = acc[i][j][4 * g + 1];
                const float v2 = acc[i][j][4 * g + 2], v3 = acc[i][j][4 * g + 3];
                if constexpr (C_F32) {
                    float* p = (float*)Cp + (int64_t)m * ldc + n;
                    if (n + 3 < N) {
                        *(float4*)p = make_float4(v0, v1, v2, v3);
                    } else {
                        if (n < N) p[0] = v0;
                        if (n + 1 < N) p[1] = v1;
                        if (n + 2 < N) p[2] = v2;
                    }
                } else {
                    bf16* p = (bf16*)Cp + (int64_t)m * ldc + n;
                    if (n + 3 < N) {
                        bf16x4 o;
                        o[0] = (bf16)v0; o[1] = (bf16)v1; o[2] = (bf16)v2; o[3] = (bf16)v3;
                        *(bf16x4*)p = o;
                    } else {
                        if (n < N) p[0] = (bf16)v0;
                        if (n + 1 < N) p[1] = (bf16)v1;
                        if (n + 2 < N) p[2] = (bf16)v2;
                    }
                }
            }
        }
    }
}

// bf16 operands, K a multiple of BK: tiles move global -> LDS on the DMA path
// (buffer_load_dwordx4 ... lds: each lane writes 16 bytes at its lane slot of a 1 KB LDS
// block), so there are no staging registers and no ds_write instructions. A lane picks
// the global chunk that belongs at its slot under the XOR swizzle. The LDS holds a ring
// of NS stages, NS-1 tiles ahead of the one being multiplied (two schedules, below). The
// DMA is issued from inline assembly
// (M0 = LDS destination) and its completion is awaited by explicit vmcnt waits, so the
// compiler does not serialise the prefetch behind each tile's LDS reads. Rows past M
// or N are clamped to a valid row (their results are never stored). Fragments of
// k-substep s+1 are read from LDS while the MFMAs of substep s run.
// WM x WN waves; with 8 waves two share each SIMD, so one wave's barrier and LDS waits
// are covered by the other's MFMAs. SPLIT: workgroup (tile, blockIdx.y) multiplies the
// K-slice [blockIdx.y * K, (blockIdx.y + 1) * K) (K is the slice length) and stores its
// fp32 partial tile at part[blockIdx.y][M][N]; a reduce kernel adds the slices.
// F32: the operands are float32 rows passed as bf16 rows of twice the length (K, lda and
// ldb in bf16 units); the DMA and the LDS layout only move bytes, and each 16-byte fragment
// (4 floats along k) feeds four v_mfma_f32_32x32x2_f32 instead of one bf16 MFMA.
// MB16: 16x16 MFMA blocks. FINE: the second, fully ordered schedule of the k loop. SB (with
// FINE): one set of weight fragments, each reloaded right after its last MFMA of a substep
// (the MFMAs run weight block by weight block), which frees registers for wider tiles.
template <int ROLE, int BM, int BN, int BK, int NS, int WM, int WN, bool C_F32, bool SPLIT = false, bool F32 = false,
          bool MB16 = false, bool FINE = false, bool SB = false>
__global__ __launch_bounds__(64 * WM * WN) void gemm_bf16_dma(int M, int N, int K, const bf16* __restrict__ A,
                                                              int64_t lda, const bf16* __restrict__ B, int64_t ldb,
                                                              void* __restrict__ Cp, int64_t ldc, int tiles_m,
                                                              int tiles_n, float* __restrict__ part) {
    constexpr int NW = WM * WN;
    constexpr int WTM = BM / WM, WTN = BN / WN;
    // MFMA blocks: 32x32 (bf16 32x32x16 or fp32 32x32x2), or 16x16 (MB16: bf16 16x16x32 or
    // fp32 16x16x4)
    constexpr int BLK = MB16 ? 16 : 32;
    constexpr int TM = WTM / BLK, TN = WTN / BLK;
    static_assert(TM * BLK == WTM && TN * BLK == WTN, "whole MFMA blocks per wave");
    using AccT = typename std::conditional<MB16, f32x4, f32x16>::type;
    constexpr int QG = MB16 ? 1 : 4;        // float4 groups of an accumulator
    constexpr int CPR = BK / 8;             // 16-byte chunks per row
    constexpr int RPB = 64 / CPR;           // rows per 1 KB DMA block
    // DMA blocks of one stage: BM / RPB activation blocks, then BN / RPB weight blocks. When
    // they split evenly, wave w takes AG consecutive activation and BG weight blocks;
    // otherwise (a 2-deep ring only, whose waits are for all of a wave's loads) block b goes to
    // wave b % NW, so waves take QM or QM - 1 blocks
    constexpr bool EVEN = BM % (RPB * NW) == 0 && BN % (RPB * NW) == 0;
    constexpr int TBA = BM / RPB, TBT = (BM + BN) / RPB, QM = (TBT + NW - 1) / NW;
    constexpr int AG = EVEN ? BM / RPB / NW : 0, BG = EVEN ? BN / RPB / NW : 0;  // DMA blocks per wave per stage
    constexpr int OPS = EVEN ? AG + BG : QM;
    constexpr int SUB = MB16 ? BK / 32 : BK / 16;  // MFMA k-substeps per stage (2 or 4 chunks of a row each)
    static_assert(NS >= 2 && BM % RPB == 0 && BN % RPB == 0, "tile");
    static_assert(EVEN ? (AG >= 1 && BG >= 1) : NS == 2, "uneven DMA blocks need the 2-deep ring");
    static_assert(SUB % 2 == 0, "fragment sets alternate within a tile");
    // one LDS block: the operand ring, reused after the k loop to stage the output tile
    constexpr int RING = NS * (BM + BN) * BK * 2;
    using OT = typename std::conditional<C_F32 || SPLIT, float, bf16>::type;
    // stage the output tile (or a K-slice's fp32 partial tile) through LDS, in one or two
    // passes of whole wave rows: whole-line stores instead of the MFMA layout's 16-byte
    // pieces spread over 32 rows
    constexpr int PASSES = (BM * BN * (int)sizeof(OT) + RING - 1) / RING;
    constexpr int RB = BM / PASSES;  // tile rows per pass
    constexpr bool STAGE = (BN * (int)sizeof(OT)) % 128 == 0 && PASSES <= 2 && BM % PASSES == 0 &&
                           RB % (BM / WM) == 0;
    __shared__ __attribute__((aligned(1024))) char smem[RING];
    bf16 (*As)[BM * BK] = reinterpret_cast<bf16 (*)[BM * BK]>(smem);
    bf16 (*Bs)[BN * BK] = reinterpret_cast<bf16 (*)[BN * BK]>(smem + NS * BM * BK * 2);

    int tm, tn;
    tile_of(tiles_m, tiles_n, tm, tn);
    const int m0 = tm * BM, n0 = tn * BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WN, wn = wave % WN;
    if constexpr (SPLIT) {
        A += (int64_t)blockIdx.y * K;
        B += (int64_t)blockIdx.y * K;
    }

    const int lr = lane / CPR, lp = lane % CPR;
    // the tile's row panels as buffer resources; a lane's chunk is a fixed byte offset in
    // them and the k advance goes in the scalar offset
    const __amdgpu_buffer_rsrc_t ra = buffer_rsrc(A + (int64_t)m0 * lda, (uint32_t)((int64_t)min(BM, M - m0) * lda * 2));
    const __amdgpu_buffer_rsrc_t rbr = buffer_rsrc(B + (int64_t)n0 * ldb, (uint32_t)((int64_t)min(BN, N - n0) * ldb * 2));
    auto a_off = [&](int r) { return (uint32_t)(((int64_t)(min(m0 + r, M - 1) - m0) * lda + swz_k<BK>(r, lp) * 8) * 2); };
    auto b_off = [&](int r) { return (uint32_t)(((int64_t)(min(n0 + r, N - 1) - n0) * ldb + swz_k<BK>(r, lp) * 8) * 2); };
    const uint32_t a_lds = (uint32_t)(uintptr_t)(lds_ptr_t)&As[0][0];
    const uint32_t b_lds = (uint32_t)(uintptr_t)(lds_ptr_t)&Bs[0][0];
    constexpr int NA = EVEN ? AG : QM, NB = EVEN ? BG : 1;
    uint32_t aoff[NA], boff[NB];
    const int wu = __builtin_amdgcn_readfirstlane(wave);  // wave-uniform, for the block choice
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
    auto dma = [&](int kt, int stage) {
        const int k0 = kt * BK;
        if constexpr (EVEN) {
#pragma unroll
            for (int q = 0; q < AG; ++q)
                dma16(ra, aoff[q], (uint32_t)k0 * 2, __builtin_amdgcn_readfirstlane(a_lds + (uint32_t)((stage * BM + (wave * AG + q) * RPB) * BK * 2)));
#pragma unroll
            for (int q = 0; q < BG; ++q)
                dma16(rbr, boff[q], (uint32_t)k0 * 2, __builtin_amdgcn_readfirstlane(b_lds + (uint32_t)((stage * BN + (wave * BG + q) * RPB) * BK * 2)));
        } else {
#pragma unroll
            for (int q = 0; q < QM; ++q) {
                const int b = wu + NW * q;
                if (b < TBA)
                    dma16(ra, aoff[q], (uint32_t)k0 * 2, a_lds + (uint32_t)((stage * BM + b * RPB) * BK * 2));
                else if (b < TBT)
                    dma16(rbr, aoff[q], (uint32_t)k0 * 2, b_lds + (uint32_t)((stage * BN + (b - TBA) * RPB) * BK * 2));
            }
        }
    };

    AccT acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = AccT{};
    // a lane's fragment rows are wm * WTM + i * BLK + lane % BLK: the block offsets are
    // multiples of 16 rows, which leave the swizzle key (row bits 1-3, or 2-3 for 32-wide
    // stages) unchanged, so block i is a constant offset from block 0 and every fragment
    // address is one per-lane base plus an immediate
    static_assert(WTM % 16 == 0 && WTN % 16 == 0 && BLK % 16 == 0, "swizzle key per lane");
    const int arow0 = wm * WTM + (lane & (BLK - 1)), brow0 = wn * WTN + (lane & (BLK - 1));
    // lane l's output columns of float4 group g of a block (its row is l % BLK): the MFMA
    // layouts with the weight fragment as the first operand
    auto ocol = [&](int g) { return MB16 ? 4 * (lane >> 4) : 8 * g + 4 * (lane >> 5); };

    const int nk = K / BK;
    bf16x8 fa[2][TM], fb[2][TN];
    auto frag = [&](int stage, int s, int set) {
        const bf16* as = As[stage];
        const bf16* bs = Bs[stage];
        const int c = MB16 ? s * 4 + (lane >> 4) : s * 2 + (lane >> 5);
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[set][i] = *(const bf16x8*)&as[(arow0 + i * BLK) * BK + swz_k<BK>(arow0, c) * 8];
#pragma unroll
        for (int j = 0; j < TN; ++j) fb[set][j] = *(const bf16x8*)&bs[(brow0 + j * BLK) * BK + swz_k<BK>(brow0, c) * 8];
    };
    auto mfma = [&](int set) {
        if constexpr (MB16 && !F32) {
            // bf16 on 16x16 blocks: lane group g = l / 16 takes chunk 4s + g, the 8 values of
            // k = 32s + 8g .. 32s + 8g + 7 that v_mfma_f32_16x16x32_bf16 expects of it
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[set][j], fa[set][i], acc[i][j], 0, 0, 0);
        } else if constexpr (MB16) {
            // float32 operands on 16x16 blocks: lane group g = l / 16 takes chunk 4s + g, so
            // MFMA u sums k = 16s + 4g + u over the four groups
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(f32x4, fb[set][j])[u],
                                                                         __builtin_bit_cast(f32x4, fa[set][i])[u],
                                                                         acc[i][j], 0, 0, 0);
        } else if constexpr (F32) {
            // float32 operands: a 16-byte chunk holds 4 floats along k; lanes 0-31 take chunk
            // 2s, lanes 32-63 chunk 2s + 1, so MFMA u sums k = 8s + u and 8s + 4 + u
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(__builtin_bit_cast(f32x4, fb[set][j])[u],
                                                                         __builtin_bit_cast(f32x4, fa[set][i])[u],
                                                                         acc[i][j], 0, 0, 0);
        } else {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[set][j], fa[set][i], acc[i][j], 0, 0, 0);
        }
    };
    // one MFMA per fragment read, then the remaining MFMAs of the substep
    constexpr int NMF = TM * TN * (F32 ? 4 : 1);
    auto interleave = [&]() {
#pragma unroll
        for (int q = 0; q < TM + TN; ++q) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        if (NMF > TM + TN) __builtin_amdgcn_sched_group_barrier(0x008, NMF - (TM + TN), 0);
    };

    if constexpr (!FINE) {
        // First schedule: the DMA of tile kt+NS-1 goes out at the top of tile kt, all at once.
#pragma unroll
        for (int st = 0; st < NS - 1; ++st)
            if (st < nk) dma(st, st);
        // tile 0 complete: NS-2 newer tiles may stay in flight, unless K has fewer tiles than that
        if (nk >= NS - 1) wait_vm<(NS - 2) * OPS>();
        else wait_vm<0>();
        __syncthreads();
        frag(0, 0, 0);
        for (int kt = 0; kt < nk; ++kt) {
            const int cur = kt % NS;
            if (kt + NS - 1 < nk) dma(kt + NS - 1, (kt + NS - 1) % NS);
            // substeps 0 .. SUB-2, each reading the fragments of the next
#pragma unroll
            for (int s = 0; s + 1 < SUB; ++s) {
                frag(cur, s + 1, (s + 1) & 1);
                mfma(s & 1);
                interleave();
            }
            // Tile kt+1 must be complete in LDS (this wave's DMA, then all waves'), and this
            // wave's reads of stage cur must be done before anyone refills it. The barrier
            // sits before the last substep so its MFMAs cover the first reads of tile kt+1.
            if (kt + 1 < nk) {
                const int newer = min(NS - 2, nk - 2 - kt);  // tiles newer than kt+1 in flight
                if (newer >= NS - 2) wait_vm<(NS - 2) * OPS>();
                else wait_vm<0>();  // tail: wait for everything
            }
            __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): fragments of the last substep are in
            __syncthreads();
            if (kt + 1 < nk) frag((kt + 1) % NS, 0, SUB & 1);
            mfma((SUB - 1) & 1);
            interleave();
        }
    } else {
    // Second schedule: every load, fragment read and MFMA in a fixed order. A stage is
    // refilled as soon as every wave has read its last fragments (at the barrier one substep
    // before the end of its tile), with the DMA blocks spread one every few MFMAs, so a wave
    // never waits behind a run of its own loads while the MFMA pipe idles.
    // One DMA block d of tile kt into stage `stage`, from resources rA / rB (the panels, or
    // empty resources: a load past the last tile then reads nothing and writes zeros into a
    // stage that is never read again, which keeps every wave's load count the same)
    auto dma_one = [&](int kt, int stage, auto D, __amdgpu_buffer_rsrc_t rA, __amdgpu_buffer_rsrc_t rB)
                       __attribute__((always_inline)) {
        constexpr int d = decltype(D)::value;
        const uint32_t k2 = (uint32_t)(kt * BK) * 2;
        if constexpr (EVEN) {
            if constexpr (d < AG)
                dma16(rA, aoff[d], k2, __builtin_amdgcn_readfirstlane(a_lds + (uint32_t)((stage * BM + (wave * AG + d) * RPB) * BK * 2)));
            else
                dma16(rB, boff[d - AG], k2, __builtin_amdgcn_readfirstlane(b_lds + (uint32_t)((stage * BN + (wave * BG + d - AG) * RPB) * BK * 2)));
        } else {
            const int b = wu + NW * d;
            if (b < TBA)
                dma16(rA, aoff[d], k2, a_lds + (uint32_t)((stage * BM + b * RPB) * BK * 2));
            else if (b < TBT)
                dma16(rB, aoff[d], k2, b_lds + (uint32_t)((stage * BN + (b - TBA) * RPB) * BK * 2));
        }
    };
    const __amdgpu_buffer_rsrc_t ra_none = buffer_rsrc(A, 0), rb_none = buffer_rsrc(B, 0);
    // every DMA block of tile kt into stage `stage` (none past the last tile)
    auto dma_all = [&](int kt, int stage) __attribute__((always_inline)) {
        const bool live = kt < nk;
        static_for<OPS>([&](auto D) __attribute__((always_inline)) {
            dma_one(kt, stage, D, live ? ra : ra_none, live ? rbr : rb_none);
        });
    };
    // fragment f (activation blocks, then weight blocks) of substep s of stage `stage`
    auto frag_one = [&](int stage, int s, auto SET, auto F) __attribute__((always_inline)) {
        constexpr int set = decltype(SET)::value, f = decltype(F)::value;
        const int c = MB16 ? s * 4 + (lane >> 4) : s * 2 + (lane >> 5);
        if constexpr (f < TM) fa[set][f] = *(const bf16x8*)&As[stage][(arow0 + f * BLK) * BK + swz_k<BK>(arow0, c) * 8];
        else fb[SB ? 0 : set][f - TM] = *(const bf16x8*)&Bs[stage][(brow0 + (f - TM) * BLK) * BK + swz_k<BK>(brow0, c) * 8];
    };
    // MFMA q of a substep (block row by block row; with SB block column by block column)
    static_assert(!F32, "the second schedule is for bf16 operands (the float32 tiles keep the first)");
    auto mfma_one = [&](auto SET, auto Q) __attribute__((always_inline)) {
        constexpr int set = decltype(SET)::value, q = decltype(Q)::value;
        constexpr int i = SB ? q % TM : q / TN, j = SB ? q / TM : q % TN, sb = SB ? 0 : set;
        if constexpr (MB16)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[sb][j], fa[set][i], acc[i][j], 0, 0, 0);
        else
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[sb][j], fa[set][i], acc[i][j], 0, 0, 0);
    };
    // one substep: the NMF MFMAs of fragment set SET, with the reads of the other set
    // (substep rsub of stage rs) and, with DMA, the OPS refill blocks of tile dkt into stage
    // dst spread evenly between them; the order is pinned, so no wave issues a run of loads
    // while its MFMAs wait
    auto substep = [&](auto DMA, auto SET, int rs, int rsub, int dkt, int dst) __attribute__((always_inline)) {
        constexpr int set = decltype(SET)::value;
        const bool live = dkt < nk;
        const __amdgpu_buffer_rsrc_t rA = live ? ra : ra_none, rB = live ? rbr : rb_none;
        static_for<NMF>([&](auto Q) __attribute__((always_inline)) {
            constexpr int q = decltype(Q)::value;
            if constexpr (decltype(DMA)::value)
                static_for<OPS>([&](auto D) __attribute__((always_inline)) {
                    if constexpr (decltype(D)::value * NMF / OPS == q) dma_one(dkt, dst, D, rA, rB);
                });
            // the next set's reads go out first, one per MFMA, so they land early (with SB the
            // weight fragments only after their last MFMA here)
            static_for<SB ? TM : TM + TN>([&](auto F) __attribute__((always_inline)) {
                if constexpr ((decltype(F)::value < NMF ? decltype(F)::value : NMF - 1) == q)
                    frag_one(rs, rsub, std::integral_constant<int, set ^ 1>{}, F);
            });
            mfma_one(SET, Q);
            if constexpr (SB && q % TM == TM - 1)
                frag_one(rs, rsub, std::integral_constant<int, set ^ 1>{}, std::integral_constant<int, TM + q / TM>{});
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    // Every wave issues OPS loads per tile for NS tiles ahead, tiles past the last included
    // (as loads of nothing), so every wait below is the same count.
    static_for<NS - 1>([&](auto ST) __attribute__((always_inline)) { dma_all(ST, ST); });
    wait_vm<(NS - 2) * OPS>();  // tile 0 complete
    dma_all(NS - 1, NS - 1);    // the last stage of the ring is free from the start
    __syncthreads();
    frag(0, 0, 0);
    for (int kt = 0; kt < nk; ++kt) {
        const int cur = kt % NS;
        // substeps 0 .. SUB-2, each reading the fragments of the next
        static_for<SUB - 1>([&](auto S) __attribute__((always_inline)) {
            constexpr int s = decltype(S)::value;
            substep(std::false_type{}, std::integral_constant<int, s & 1>{}, cur, s + 1, 0, 0);
        });
        // Tile kt+1 must be complete in LDS (this wave's DMA, then all waves'), and every
        // wave's reads of stage cur must be done before it is refilled. The barrier sits
        // before the last substep, so its MFMAs cover the first reads of tile kt+1, and the
        // refill of stage cur with tile kt+NS goes out between them: each tile's DMA has a
        // whole tile of MFMAs, from one barrier to the next, to land. (After the last tile
        // the reads of stage (kt+1) % NS fetch values that are never used.)
        wait_vm<(NS - 2) * OPS>();
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): fragments of the last substep are in
        __syncthreads();
        substep(std::true_type{}, std::integral_constant<int, (SUB - 1) & 1>{}, (kt + 1) % NS, 0, kt + NS, cur);
    }
    wait_vm<0>();  // the loads of nothing past the last tile write the ring too
    }

    if constexpr (STAGE) {
        // tile row r is stored as 16-byte chunks, chunk c at position c ^ (r & 7)
        constexpr int E16 = 16 / (int)sizeof(OT);   // elements per chunk
        constexpr int CPR_O = BN / E16;             // chunks per tile row
        OT* st = reinterpret_cast<OT*>(smem);
        // a K-slice's fp32 partial goes to part[blockIdx.y] (row stride N), the output to C
        OT* const out = SPLIT ? reinterpret_cast<OT*>(part + (int64_t)blockIdx.y * M * N) : (OT*)Cp;
        const int64_t ldo = SPLIT ? (int64_t)N : ldc;
        const bool vec = ((uintptr_t)out & 15) == 0 && (ldo * (int64_t)sizeof(OT)) % 16 == 0;
#pragma unroll
        for (int pass = 0; pass < PASSES; ++pass) {
            __syncthreads();  // every wave is done with the ring (then with the previous pass)
            if (wm * WTM >= pass * RB && wm * WTM < (pass + 1) * RB) {
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    const int r = wm * WTM - pass * RB + i * BLK + (lane & (BLK - 1));
#pragma unroll
                    for (int j = 0; j < TN; ++j)
#pragma unroll
                        for (int g = 0; g < QG; ++g) {
                            const int col = wn * WTN + j * BLK + ocol(g);
                            OT* q = st + r * BN + (((col / E16) ^ (r & 7)) * E16) + col % E16;
                            const float v0 = acc[i][j][4 * g], v1 = acc[i][j][4 * g + 1];
                            const float v2 = acc[i][j][4 * g + 2], v3 = acc[i][j][4 * g + 3];
                            if constexpr (sizeof(OT) == 4) {
                                *(float4*)q = make_float4(v0, v1, v2, v3);
                            } else {
                                bf16x4 o;
                                o[0] = (bf16)v0; o[1] = (bf16)v1; o[2] = (bf16)v2; o[3] = (bf16)v3;
                                *(bf16x4*)q = o;
                            }
                        }
                }
            }
            __syncthreads();
            for (int c = tid; c < RB * CPR_O; c += 64 * NW) {
                const int r = c / CPR_O, cc = c % CPR_O;
                const int m = m0 + pass * RB + r, n = n0 + cc * E16;
                if (m >= M || n >= N) continue;
                const OT* q = st + r * BN + ((cc ^ (r & 7)) * E16);
                OT* p = out + (int64_t)m * ldo + n;
                if (vec && n + E16 <= N) {
                    *(u32x4*)p = *(const u32x4*)q;
                } else {
                    for (int e = 0; e < E16 && n + e < N; ++e) p[e] = q[e];
                }
            }
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int m = m0 + wm * WTM + i * BLK + (lane & (BLK - 1));
        if (m >= M) continue;
#pragma unroll
        for (int j = 0; j < TN; ++j) {
#pragma unroll
            for (int g = 0; g < QG; ++g) {
                const int n = n0 + wn * WTN + j * BLK + ocol(g);
                const float v0 = acc[i][j][4 * g], v1 = acc[i][j][4 * g + 1];
                const float v2 = acc[i][j][4 * g + 2], v3 = acc[i][j][4 * g + 3];
                if constexpr (SPLIT) {
                    float* p = part + ((int64_t)blockIdx.y * M + m) * N + n;
                    if (n + 3 < N && (N & 3) == 0) {
                        *(float4*)p = make_float4(v0, v1, v2, v3);
                    } else {
                        if (n < N) p[0] = v0;
                        if (n + 1 < N) p[1] = v1;
                        if (n + 2 < N) p[2] = v2;
                        if (n + 3 < N) p[3] = v3;
                    }
                } else if constexpr (C_F32) {
                    float* p = (float*)Cp + (int64_t)m * ldc + n;
                    if (n + 3 < N) {
                        *(float4*)p = make_float4(v0, v1, v2, v3);
                    } else {
                        if (n < N) p[0] = v0;
                        if (n + 1 < N) p[1] = v1;
                        if (n + 2 < N) p[2] = v2;
                    }
                } else {
                    bf16* p = (bf16*)Cp + (int64_t)m * ldc + n;
                    if (n + 3 < N) {
                        bf16x4 o;
                        o[0] = (bf16)v0; o[1] = (bf16)v1; o[2] = (bf16)v2; o[3] = (bf16)v3;
                        *(bf16x4*)p = o;
                    } else {
                        if (n < N) p[0] = (bf16)v0;
                        if (n + 1 < N) p[1] = (bf16)v1;
                        if (n + 2 < N) p[2] = (bf16)v2;
                    }
                }
            }
        }
    }
}

// C[m][n] = sum over the slices, in slice order, of part[slice][m][n]; 4 outputs per thread
template <bool C_F32>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const float* __restrict__ part, int splits, int M, int N,
                                                            void* __restrict__ Cp, int64_t ldc) {
    const int n4 = (N + 3) / 4;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (int64_t)M * n4) return;
    const int m = (int)(i / n4), n = (int)(i % n4) * 4;
    const int64_t slice = (int64_t)M * N;
    const float* p = part + (int64_t)m * N + n;
    float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    const bool full = n + 3 < N && (N & 3) == 0;
    for (int sp = 0; sp < splits; ++sp, p += slice) {
        if (full) {
            const float4 q = *(const float4*)p;
            v[0] += q.x; v[1] += q.y; v[2] += q.z; v[3] += q.w;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (n + e < N) v[e] += p[e];
        }
    }
    if constexpr (C_F32) {
        float* c = (float*)Cp + (int64_t)m * ldc + n;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (n + e < N) c[e] = v[e];
    } else {
        bf16* c = (bf16*)Cp + (int64_t)m * ldc + n;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (n + e < N) c[e] = (bf16)v[e];
    }
}

template <int ROLE, int BM, int BN, int BK, int NS, int WM, int WN, bool CF, bool MB16 = false, bool FINE = false,
          bool SB = false>
hipError_t run_dma(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const void* B, int64_t ldb, void* C,
                   int64_t ldc, hipStream_t s, int splits = 1, float* part = nullptr) {
    const int tm = (int)((M + BM - 1) / BM), tn = (int)((N + BN - 1) / BN);
    if (splits <= 1 && !C) return hipErrorInvalidValue;
    if (splits <= 1) {
        SSM_LAUNCH((gemm_bf16_dma<ROLE, BM, BN, BK, NS, WM, WN, CF, false, false, MB16, FINE, SB>), dim3(tm * tn), dim3(64 * WM * WN), 0, s,
                   (int)M, (int)N, (int)K, (const bf16*)A, lda, (const bf16*)B, ldb, C, ldc, tm, tn, nullptr);
        return hipGetLastError();
    }
    // K-slices are built for the tiles that pick_tile slices
    if constexpr (BK == 64 && BM * BN <= 192 * 128 && BM != 96) {
        SSM_LAUNCH((gemm_bf16_dma<ROLE, BM, BN, BK, NS, WM, WN, CF, true, false, MB16, FINE, SB>), dim3(tm * tn, splits), dim3(64 * WM * WN), 0,
                   s, (int)M, (int)N, (int)(K / splits), (const bf16*)A, lda, (const bf16*)B, ldb, C, ldc, tm, tn, part);
        if (const hipError_t e = hipGetLastError(); e != hipSuccess) return e;
        if (!C) return hipSuccess;  // the caller takes the partials
        KernelTimer kt("gemm.splitk_reduce", s);
        const int64_t n = M * ((N + 3) / 4);
        SSM_LAUNCH((splitk_reduce_kernel<CF>), dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, (const float*)part,
                   splits, (int)M, (int)N, C, ldc);
        return hipGetLastError();
    }
    return hipErrorInvalidValue;
}

hipError_t reduce_slices_f32(const float* part, int splits, int64_t M, int64_t N, float* C, int64_t ldc, hipStream_t s) {
    KernelTimer kt("gemm.splitk_reduce", s);
    const int64_t n4 = M * ((N + 3) / 4);
    SSM_LAUNCH((splitk_reduce_kernel<true>), dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, s, part, splits, (int)M,
               (int)N, C, ldc);
    return hipGetLastError();
}

// float32 operands on the DMA tiles: the rows are moved as bytes, so the kernel sees them as
// bf16 rows of twice the length (K, lda, ldb doubled); only the MFMAs read them as floats
template <int ROLE, int BM, int BN, int NS, int WM, int WN, bool MB16 = false>
hipError_t run_dma_f32(int64_t M, int64_t N, int64_t K, const float* A, int64_t lda, const float* B, int64_t ldb,
                       float* C, int64_t ldc, hipStream_t s, int splits = 1, float* part = nullptr) {
    const int tm = (int)((M + BM - 1) / BM), tn = (int)((N + BN - 1) / BN);
    if (splits <= 1) {
        SSM_LAUNCH((gemm_bf16_dma<ROLE, BM, BN, 64, NS, WM, WN, true, false, true, MB16>), dim3(tm * tn), dim3(64 * WM * WN),
                   0, s, (int)M, (int)N, (int)(2 * K), (const bf16*)A, 2 * lda, (const bf16*)B, 2 * ldb, C, ldc, tm,
                   tn, nullptr);
        return hipGetLastError();
    }
    SSM_LAUNCH((gemm_bf16_dma<ROLE, BM, BN, 64, NS, WM, WN, true, true, true, MB16>), dim3(tm * tn, splits),
               dim3(64 * WM * WN), 0, s, (int)M, (int)N, (int)(2 * K / splits), (const bf16*)A, 2 * lda,
               (const bf16*)B, 2 * ldb, C, ldc, tm, tn, part);
    if (const hipError_t e = hipGetLastError(); e != hipSuccess) return e;
    return reduce_slices_f32(part, splits, M, N, C, ldc, s);
}

// bf16 tiles. Which one is fastest depends on how many of them the output gives: an MI355X
// runs 256 workgroups at a time (one per CU; the two smallest tiles' rings fit a CU twice), and
// a part-empty round costs as much as a full one. Every tile is therefore priced as
//   launch + rounds x (a x (64-wide k-tiles) + b)
// with a and b (us) fitted to its own measured times over 647 shapes, M = 80 .. 65536,
// N = 80 .. 16384 and K = 384 .. 8192, weights read from memory; a is what a k-tile costs on a
// CU that holds one tile (6.8 TFLOP/s per CU for 256x320, 4.4 for 128x128, 1.9 for 64x64: bytes
// moved per flop), b the first loads' latency and the store. The cheapest is within 2% of the
// best tile on average over those shapes (6% at the 90th percentile). It knows no memory rate: a product
// bound by reading A (65536x288x2048, 268 MB) takes longer than its price (100 us, priced 58), and the
// tile of least price is the fastest there too (the others 105-136). Against the rule before
// it (128x128 with a 2-deep ring, 256x256, 256x320 when N is a multiple of 320, and the decode
// tile kernel up to 512 rows): 391x10240x2560 54.7 -> 30.9 us, 391x2560x5120 36.8 -> 25.3,
// 1024x3584x3584 47.0 -> 32.9, 2048x2560x5120 85.0 -> 56.1, 2048x5120x2560 88.2 -> 52.0,
// 4096x2560x5120 153.9 -> 94.3, 2900x4096x8192 202 -> 153, 65536x2560x5120 1303 -> 1223 us. A ring of 3 or 4 stages is worth more than a second workgroup
// per CU on a grid that gives each CU one tile (128x128, 3-deep against 2-deep: 0.48 against
// 0.75 us per k-tile).
enum BfTile {
    kT32x64, kT64x64, kT64x128, kT96x128, kT128x128, kT128x192, kT192x128, kT128x256, kT256x128, kT256x192, kT192x256,
    kT256x256, kT256x320, kBfTiles
};
struct TileCost {
    int bm, bn;
    float a, a2, b;  // a2: per k-tile when two tiles share a CU (0: the ring fills it)
    bool split;      // K-slices of it are built
};
constexpr TileCost kTileCost[kBfTiles] = {
    {32, 64, 0.186f, 0.243f, 1.06f, true}, {64, 64, 0.278f, 0.381f, 0.84f, true}, {64, 128, 0.321f, 0.0f, 1.50f, true},
    {96, 128, 0.405f, 0.0f, 2.55f, false}, {128, 128, 0.480f, 0.0f, 1.36f, true}, {128, 192, 0.633f, 0.0f, 2.48f, true},
    {192, 128, 0.603f, 0.0f, 2.55f, true}, {128, 256, 0.786f, 0.0f, 2.74f, false}, {256, 128, 0.748f, 0.0f, 3.25f, false},
    {256, 192, 1.087f, 0.0f, 2.76f, false}, {192, 256, 1.111f, 0.0f, 2.07f, false}, {256, 256, 1.336f, 0.0f, 3.01f, false},
    {256, 320, 1.554f, 0.0f, 6.65f, false}};
constexpr int kMaxSlices = 8, kMinSliceK = 8;  // K-slices: at most 8, of at least 8 k-tiles each
constexpr float kLaunchUs = 2.0f;

// Past four rounds the two widest tiles are set against each other by whole rounds, 256x320 priced 4%
// higher: those grids stay in step (all workgroups take the same time), and its price comes out low there.
// 256x256 against 256x320, us: 65536x4096x4096 1567 and 1577 (16 rounds, 13); 32768x5376x2688 743 and 763
// (11, 9); 14384x10240x5120 1118 and 1170 (9, 8); 65536x2560x2560 684 and 696 (10, 8); 16384x10240x5120
// 1285 and 1245 (10, 8); 20480x5120x2560 429 and 404 (7, 5); 40000x5120x2560 857 and 822 (13, 10). Up to four
// rounds the price holds as it is (16384x5120x2560 310 and 308, 14384x5120x2560 301 and 295, 16384x2560x2560
// 178 and 155).
constexpr float kWidePrice = 1.04f;

struct GemmPlan {
    int tile;    // BfTile, or -1: the few-row / decode tile kernels
    int slices;  // K-slices (1: none)
    float us;    // its price
};

// after a few rounds the workgroups no longer run in step: the last round costs about its share
float rounds_of(int64_t wg) { return wg <= 4 * 256 ? (float)((wg + 255) / 256) : (float)wg / 256.0f + 0.6f; }

float tile_us(const TileCost& t, int64_t wg, float nk) {
    const float r = rounds_of(wg);
    if (t.a2 > 0.0f && wg > 256) return kLaunchUs + (float)((wg + 511) / 512) * t.a2 * nk + r * t.b;
    return kLaunchUs + r * (t.a * nk + t.b);
}

// the cheapest tile (and K-slice count within the scratch) for C[M][N] = A[M][K] B[N][K]^T,
// K a multiple of 64
GemmPlan pick_tile(int64_t M, int64_t N, int64_t K, size_t scratch_bytes) {
    GemmPlan best{kT64x64, 1, 1e30f};
    const int64_t nk = K / 64;
    for (int i = 0; i < kBfTiles; ++i) {
        const TileCost& t = kTileCost[i];
        const int64_t tiles = ((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn);
        const float u = tile_us(t, tiles, (float)nk);
        bool less = u < best.us;
        if (i == kT256x320 && tiles > 4 * 256) {
            const TileCost& q = kTileCost[kT256x256];
            const int64_t r = (tiles + 255) / 256, rq = (((M + 255) / 256) * ((N + 255) / 256) + 255) / 256;
            less = best.tile == kT256x256 ? kWidePrice * (float)r * (t.a * (float)nk + t.b) < (float)rq * (q.a * (float)nk + q.b)
                                          : kWidePrice * u < best.us;
        }
        if (less) best = GemmPlan{i, 1, u};
        if (!t.split || tiles >= 192) continue;
        for (int d = 2; d <= kMaxSlices && d * kMinSliceK <= nk && tiles * d <= 288; ++d) {
            const size_t bytes = (size_t)d * M * N * 4;
            if (nk % d != 0 || bytes > scratch_bytes) continue;
            const float us = tile_us(t, tiles * d, (float)(nk / d)) + split_reduce_us(bytes);
            if (us < best.us) best = GemmPlan{i, d, us};
        }
    }
    return best;
}

// Float32 tiles by the same kind of model: rounds of workgroups (one per CU; two for the 64 KB
// ring of 128x128) times the work a CU does per round over the tile's measured per-CU MFMA
// efficiency. On the hybrid shard's 2048-row chunks: 256x256 tiles (8 waves of 128x64) 0.91,
// 256x224 (8 waves of 32x224) 0.93, 128x224 (8 waves of 32x112 on 16x16 blocks) 0.91,
// 128x128 (8 waves of 64x32, two per CU) 0.89. The 224-wide tiles exist for outputs whose
// 256-wide tiles leave part of a round empty: in_proj (2048 x 7168) takes 256 tiles of 256x224
// where 256x256 gave 224 (840 -> 720 us), out_proj (2048 x 3584) 256 tiles of 128x224 where
// 128x128 gave 448 over two slots per CU (430 -> 368 us; 4 waves of 32x224, one per SIMD,
// took 393 us; 64x112 wave tiles on 16x16 blocks for 256x224 spill).
enum F32Tiles { kF32Tiles128 = 0, kF32Tiles256 = 1, kF32Tiles256x224 = 2, kF32Tiles128x224 = 3, kF32Tiles64 = 4 };
F32Tiles f32_tiles(int64_t M, int64_t N) {
    auto cost = [&](int bm, int bn, int per_cu, double eff) {
        const int64_t tiles = ((M + bm - 1) / bm) * ((N + bn - 1) / bn), slots = 256 * per_cu;
        return (double)((tiles + slots - 1) / slots) * per_cu * bm * bn / eff;
    };
    F32Tiles best = kF32Tiles128;
    double c = cost(128, 128, 2, 0.89);
    const double c256 = cost(256, 256, 1, 0.91), c224 = cost(256, 224, 1, 0.93), c128x224 = cost(128, 224, 1, 0.91);
    if (c256 < c) { c = c256; best = kF32Tiles256; }
    if (c224 < c) { c = c224; best = kF32Tiles256x224; }
    if (c128x224 < c) { c = c128x224; best = kF32Tiles128x224; }
    return best;
}

// Time of a float32 product without the bf16 cores, in us: the same model (614 GFLOP/s of float32
// MFMA per CU) from 256 128x128 tiles on; below that the register-staged 64x64 tiles, one per CU at a
// time (measured 0.53-0.64 us per 32 k), or two K-slices of 64x64 DMA tiles, two per CU (1.0-1.1 us)
float f32_us(int64_t M, int64_t N, int64_t K, int slices) {
    const int64_t t64 = ((M + 63) / 64) * ((N + 63) / 64), t128 = ((M + 127) / 128) * ((N + 127) / 128);
    if (slices > 1) return 8.0f + (float)((t64 * slices + 511) / 512) * 1.07f * (float)(K / (32 * slices));
    if (t128 < 256) return 4.0f + (float)((t64 + 255) / 256) * 0.57f * (float)(K / 32);
    const int bm[] = {128, 256, 256, 128}, bn[] = {128, 256, 224, 224};
    const double eff[] = {0.89, 0.91, 0.93, 0.91};
    const F32Tiles t = f32_tiles(M, N);
    const int64_t tiles = ((M + bm[t] - 1) / bm[t]) * ((N + bn[t] - 1) / bn[t]);
    const int per_cu = t == kF32Tiles128 ? 2 : 1;
    const double rounds = (double)((tiles + 256 * per_cu - 1) / (256 * per_cu));
    return 5.0f + (float)(rounds * per_cu * bm[t] * bn[t] * 2.0 * K / (eff[t] * 614.4e3));
}

// Decode batches above the few-row kernels (65..512 rows) with bf16 output: the streamed
// tile kernel of the decode projections (launch_gemm_skinny) when its tiles give at least
// 128 workgroups, without K-slices
bool decode_tiles(int64_t M, int64_t N, int64_t K) {
    return K % 64 == 0 && M > 64 && M <= 512 && ((M + 31) / 32) * ((N + 31) / 32) >= 128;
}
// ... and its price in pick_tile's terms: the tile that launch_dtile_pick takes, fitted on 191 shapes
// (66 .. 512 rows, K = 768 .. 8192, median error 3.5%); a k-tile costs more the more CUs are busy. The
// choice between the two by price is within 0.2% of the faster one on average over them: 80x2560x2560
// 9.1 us here and 11.0 on the DMA tiles, 100x2048x4096 8.8 and 12.8, 140x2560x5120 13.5 and 19.3, 258x2560x5120
// 17.4 and 22.6; 391x2560x2560 19.2 and 15.9.
float decode_tile_us(int64_t M, int64_t N, int64_t K) {
    const int64_t tm64 = (M + 63) / 64, tm32 = (M + 31) / 32, tn64 = (N + 63) / 64, tn32 = (N + 31) / 32;
    auto price = [&](int64_t wg, float launch, float first, float tile, float busy) {
        const float occ = (float)std::min<int64_t>(wg, 256) / 256.0f;
        return launch + rounds_of(wg) * (first + (tile + busy * occ) * (float)(K / 64));
    };
    if (M > 128 && tm64 * tn64 >= 128) return price(tm64 * tn64, 2.07f, 1.89f, 0.128f, 0.036f);
    if (tm64 * tn32 >= 128) return price(tm64 * tn32, 1.29f, 1.70f, 0.077f, 0.035f);
    return price(tm32 * tn32, 1.23f, 1.23f, 0.100f, 0.017f);
}
// x_proj of up to 512 rows (at most 512 columns): 16-row tiles of the few-row kernel, which
// spread over more workgroups than the DMA tiles and need no K-slices. Every wave streams its
// share of K for one 16x16 tile: 192 columns, K = 1280 / 2560 / 5120 at 256 rows 4.6 / 6.9 /
// 11.7 us (DMA tiles 6.6 / 8.3 / 10.2), at 391 rows (a second round) 7.2 / 11.4 / 20.7
// (6.6 / 8.5 / 10.3).
bool xproj_decode_skinny(int64_t M, int64_t N) { return M <= 512 && N <= 512; }
float xproj_skinny_us(int64_t M, int64_t N, int64_t K) {
    return 2.0f + rounds_of(((M + 15) / 16) * ((N + 15) / 16)) * 0.122f * (float)(K / 64);
}

template <bool CF> GemmPlan plan_bf16(GemmRole role, int64_t M, int64_t N, int64_t K, size_t scratch_bytes) {
    GemmPlan p = pick_tile(M, N, K, scratch_bytes);
    float few = 1e30f;
    if (CF && role == kGemmXProj && xproj_decode_skinny(M, N)) few = xproj_skinny_us(M, N, K);
    if (!CF && decode_tiles(M, N, K)) few = decode_tile_us(M, N, K);
    if (few < p.us) p = GemmPlan{-1, 1, few};
    return p;
}

template <int ROLE, bool CF>
hipError_t dispatch_dma(const GemmPlan& g, int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const void* B,
                        int64_t ldb, void* C, int64_t ldc, hipStream_t s, float* scratch) {
#define SSM_TILE(T, BM, BN, NS, WM, WN, SB)                                                                  \
    case T: return run_dma<ROLE, BM, BN, 64, NS, WM, WN, CF, true, true, SB>(M, N, K, A, lda, B, ldb, C, ldc, s, \
                                                                             g.slices, scratch)
    switch (g.tile) {
        SSM_TILE(kT32x64, 32, 64, 6, 1, 4, false);
        SSM_TILE(kT64x64, 64, 64, 4, 2, 2, false);
        SSM_TILE(kT64x128, 64, 128, 4, 2, 4, false);
        SSM_TILE(kT96x128, 96, 128, 4, 2, 2, false);
        SSM_TILE(kT128x128, 128, 128, 3, 2, 4, false);
        SSM_TILE(kT128x192, 128, 192, 3, 2, 4, false);
        SSM_TILE(kT192x128, 192, 128, 3, 2, 4, false);
        SSM_TILE(kT128x256, 128, 256, 3, 2, 4, false);
        SSM_TILE(kT256x128, 256, 128, 3, 4, 2, false);
        SSM_TILE(kT256x192, 256, 192, 2, 4, 2, false);
        SSM_TILE(kT192x256, 192, 256, 2, 2, 4, false);
        SSM_TILE(kT256x256, 256, 256, 2, 2, 4, false);
        // one set of weight fragments: two sets of its 64x160 wave tiles do not fit the registers
        SSM_TILE(kT256x320, 256, 320, 2, 4, 2, true);
    }
#undef SSM_TILE
    return hipErrorInvalidValue;
}

// K a multiple of 32 only, or a K of few 64-wide tiles (dt_proj: K = dt_rank): 32-wide stages,
// whose rings stay small enough for several workgroups per CU; the many short-lived tiles hide
// each other's first loads. 64x64 tiles while they fit two rounds (256x3584x224 5.9 -> 4.1 us,
// 256x2560x160 5.2 -> 3.6). Above that the last round decides: 128x128 with a 4-deep ring runs 512 at
// a time, with a 3-deep ring 768, 256x128 512 (of twice the output). By 305 shapes of K = 32 .. 256, us,
// the 4-deep, 256x128 and the 3-deep:
//   up to 512 128x128 tiles the 4-deep ring (K = 160, 440 tiles 8.0 / 8.5 / 8.4);
//   up to 768 the 3-deep one (K = 96, 516 8.7 / 8.8 / 7.9);
//   then 256x128 where its last round is at least half full (K = 224, 981 18.3 / 15.3 / 16.6; K = 128, 1024
//   12.5 / 12.0 / 13.1), the 3-deep ring where it is emptier (K = 96, 2200 20.1 / 21.6 / 18.8; K = 64, 1152 12.4
//   / 13.7 / 11.5), for a shorter K up to more rounds (K = 64, 5640 256x128 37.9, 3-deep 34.7; K = 96, 5380 40.1 and
//   37.6; K = 224, 4360 47.0 and 49.8), and past those 256x128 (K = 96, 11500 97 and 122; 65536x2560x160 113 and 129).
bool dma32_deep(int64_t K, int64_t t128, float r) {  // r: rounds of 256x128
    if (t128 <= 768) return true;
    if (r <= 1.0f) return false;
    if (r <= 2.0f) return r <= (K <= 160 ? 1.5f : 1.25f);
    return r <= (K <= 96 ? 6.4f : K <= 160 ? 3.75f : 2.15f);
}

// Two kinds of K of whole 64-wide tiles do better with those (372 shapes, M = 65 .. 32768, K = 64 .. 256):
// outputs that give the few-row kernel one round of 32x32 tiles (2.7-2.9 us at K = 64 .. 256 against
// 3.0-3.8), from K = 192 on also of 64x32 (3.4-3.6 against 3.5-3.9); and from K = 192 on outputs that fill
// one round of 256x256 tiles (K = 256: 224 .. 256 tiles 13.9-15.1 us against 15.1-16.7, 192 tiles 13.3-13.5
// against 13.0-13.1; K = 192: 12.8-13.9 against 13.1-14.5).
bool dt_few_rows(int64_t M, int64_t N, int64_t K) {
    const int64_t tm64 = (M + 63) / 64, tn32 = (N + 31) / 32;
    if (!decode_tiles(M, N, K) || (M > 128 && tm64 * ((N + 63) / 64) >= 128)) return false;
    return tm64 * tn32 < 128 || (K >= 192 && tm64 * tn32 <= 256);
}
bool dt_one_round(int64_t M, int64_t N, int64_t K) {
    const int64_t tiles = ((M + 255) / 256) * ((N + 255) / 256);
    return K % 64 == 0 && K >= 192 && tiles > 204 && tiles <= 256;
}

template <int ROLE, bool CF>
hipError_t dispatch_dma32(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const void* B, int64_t ldb,
                          void* C, int64_t ldc, hipStream_t s) {
    if (((M + 63) / 64) * ((N + 63) / 64) <= 512)
        return run_dma<ROLE, 64, 64, 32, 4, 2, 2, CF>(M, N, K, A, lda, B, ldb, C, ldc, s);
    const int64_t t128 = ((M + 127) / 128) * ((N + 127) / 128);
    if (t128 <= 512) return run_dma<ROLE, 128, 128, 32, 4, 2, 4, CF>(M, N, K, A, lda, B, ldb, C, ldc, s);
    if (dma32_deep(K, t128, (float)(((M + 255) / 256) * ((N + 127) / 128)) / 512.0f))
        return run_dma<ROLE, 128, 128, 32, 3, 2, 2, CF>(M, N, K, A, lda, B, ldb, C, ldc, s);
    return run_dma<ROLE, 256, 128, 32, 3, 4, 2, CF>(M, N, K, A, lda, B, ldb, C, ldc, s);
}

// Scratch that a product may use for K-slices in a prefill of up to M rows: what kMaxSlices
// slices need, up to what the largest grid of K-slices (288 tiles of 192x128) holds.
// Monotone in M, so a workspace for more rows serves fewer.
size_t splitk_reserve(int64_t M, int64_t N) {
    return M <= 64 ? 0 : std::min((size_t)kMaxSlices * M * N * 4, (size_t)288 * 192 * 128 * 4);
}

// fp32 weights and at most 8 activation rows (a decode step of the fp32 configuration),
// where the time is the weight read: one weight row per wave, streamed in 1 KB runs (64
// lanes x 4 floats, whole cache lines) and multiplied by the activation rows (M x K floats,
// shared by every wave and served from cache); the lanes' sums meet by xor shuffles. K,
// the leading dimensions and the pointers are multiples of 4 floats (checked by the caller).
template <int ROLE>
__global__ __launch_bounds__(256) void gemv_f32_kernel(int M, int N, int K, const float* __restrict__ A,
                                                       int64_t lda, const float* __restrict__ B, int64_t ldb,
                                                       float* __restrict__ C, int64_t ldc) {
    constexpr int MR = 8;
    const int lane = threadIdx.x & 63;
    const int n = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (n >= N) return;
    const float* brow = B + (int64_t)n * ldb;
    float acc[MR];
#pragma unroll
    for (int m = 0; m < MR; ++m) acc[m] = 0.0f;
    // four 1 KB runs per iteration, so that their loads are in flight together
    for (int k0 = lane * 4; k0 < K; k0 += 1024) {
        float4 b[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            b[j] = k0 + 256 * j < K ? *(const float4*)(brow + k0 + 256 * j) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int m = 0; m < MR; ++m) {
            if (m < M) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    if (k0 + 256 * j < K) {
                        const float4 a = *(const float4*)(A + (int64_t)m * lda + k0 + 256 * j);
                        acc[m] += a.x * b[j].x + a.y * b[j].y + a.z * b[j].z + a.w * b[j].w;
                    }
                }
            }
        }
    }
    float mine = 0.0f;
#pragma unroll
    for (int m = 0; m < MR; ++m) {
        if (m < M) {
            float v = acc[m];
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
            if (lane == m) mine = v;
        }
    }
    if (lane < M) C[(int64_t)lane * ldc + n] = mine;
}

// fp32 operands on v_mfma_f32_16x16x4_f32: 64x64 tiles, k 16 per stage, four waves of 32x32.
constexpr int kFBK = 16;
constexpr int kFPad = kFBK + 1;

template <int ROLE>
__global__ __launch_bounds__(256) void gemm_f32_nt(int M, int N, int K, const float* __restrict__ A,
                                                   int64_t lda, const float* __restrict__ B, int64_t ldb,
                                                   float* __restrict__ C, int64_t ldc, int tiles_m, int tiles_n) {
    __shared__ float As[2][64 * kFPad];
    __shared__ float Bs[2][64 * kFPad];
    int tm, tn;
    tile_of(tiles_m, tiles_n, tm, tn);
    const int m0 = tm * 64, n0 = tn * 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int lrow = tid >> 2, lck = tid & 3;  // one float4 of A and of B per thread
    float4 ra, rb;
    auto gload = [&](int k0) {
        const int gk = k0 + lck * 4;
        const int gm = m0 + lrow, gn = n0 + lrow;
        ra = (gm < M && gk < K) ? *(const float4*)(A + (int64_t)gm * lda + gk) : make_float4(0, 0, 0, 0);
        rb = (gn < N && gk < K) ? *(const float4*)(B + (int64_t)gn * ldb + gk) : make_float4(0, 0, 0, 0);
    };
    auto lstore = [&](int buf) {
        float* a = &As[buf][lrow * kFPad + lck * 4];
        float* b = &Bs[buf][lrow * kFPad + lck * 4];
        a[0] = ra.x; a[1] = ra.y; a[2] = ra.z; a[3] = ra.w;
        b[0] = rb.x; b[1] = rb.y; b[2] = rb.z; b[3] = rb.w;
    };
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{};
    const int nk = (K + kFBK - 1) / kFBK;
    gload(0);
    lstore(0);
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
        const int cur = kt & 1;
        if (kt + 1 < nk) gload((kt + 1) * kFBK);
#pragma unroll
        for (int s = 0; s < kFBK / 4; ++s) {
            float af[2], bfv[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) af[i] = As[cur][(wm * 32 + i * 16 + (lane & 15)) * kFPad + s * 4 + (lane >> 4)];
#pragma unroll
            for (int j = 0; j < 2; ++j) bfv[j] = Bs[cur][(wn * 32 + j * 16 + (lane & 15)) * kFPad + s * 4 + (lane >> 4)];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(bfv[j], af[i], acc[i][j], 0, 0, 0);
        }
        if (kt + 1 < nk) lstore(cur ^ 1);
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int m = m0 + wm * 32 + i * 16 + (lane & 15);
        if (m >= M) continue;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int n = n0 + wn * 32 + j * 16 + 4 * (lane >> 4);
            float* p = C + (int64_t)m * ldc + n;
            if (n + 3 < N) {
                *(float4*)p = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
            } else {
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (n + v < N) p[v] = acc[i][j][v];
            }
        }
    }
}

// float32 k stages: 32 floats, one 128-byte line of every operand row
constexpr int kF32BK = 32;

// K-slices for a float32 product with few 128x128 tiles: the most slices (dividing the
// 32-wide stages, at least 4 stages each) that keep the grid within about two workgroups
// per CU. 1 = unsplit.
int f32_slices(int64_t tiles, int64_t K) {
    if (K % kF32BK != 0 || tiles >= 256) return 1;
    const int64_t nk = K / kF32BK, cap = std::max<int64_t>(1, 512 / tiles);
    int best = 1;
    for (int64_t d = 2; d <= cap && d <= nk / 4; ++d)
        if (nk % d == 0) best = (int)d;
    return best;
}

int fit_slices(int sp, int64_t M, int64_t N, size_t scratch_bytes) {
    return (sp > 1 && (size_t)sp * M * N * 4 <= scratch_bytes) ? sp : 1;
}

template <int ROLE, int BM, int BN, int WM, int WN, bool AF, bool CF>
hipError_t run_bf16(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const void* B, int64_t ldb,
                    void* C, int64_t ldc, hipStream_t s) {
    const int tm = (int)((M + BM - 1) / BM), tn = (int)((N + BN - 1) / BN);
    SSM_LAUNCH((gemm_bf16_nt<ROLE, BM, BN, WM, WN, AF, CF>), dim3(tm * tn), dim3(256), 0, s, (int)M, (int)N,
                       (int)K, A, lda, (const bf16*)B, ldb, C, ldc, tm, tn);
    return hipGetLastError();
}

// o[m][k] = bf16(a[m][k]) (round to nearest even), 8 values per thread; K % 8 == 0
__global__ __launch_bounds__(256) void round_bf16_rows_kernel(const float* __restrict__ a, int64_t lda,
                                                              bf16* __restrict__ o, int64_t M, int K) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int kg = K / 8;
    if (i >= M * kg) return;
    const int64_t m = i / kg;
    const int k = (int)(i % kg) * 8;
    const float* p = a + m * lda + k;
    *(bf16x8*)(o + m * K + k) = cvt8(*(const float4*)p, *(const float4*)(p + 4));
}

template <int ROLE, bool AF, bool CF>
hipError_t dispatch_bf16(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const void* B, int64_t ldb,
                         void* C, int64_t ldc, hipStream_t s, float* scratch, size_t scratch_bytes) {
    auto few_rows = [&]() {
        SkinnyArgs p{};
        p.A = A; p.lda = lda; p.a_f32 = AF; p.B = (const bf16*)B; p.ldb = ldb; p.C = C; p.ldc = ldc;
        p.M = (int)M; p.N = (int)N; p.K = (int)K;
        return launch_gemm_skinny(p, CF ? kSkinnyStoreF32 : kSkinnyStoreBf16, s);
    };
    // few rows: the weight read dominates; stream it with many narrow workgroups. fp32-A
    // dt_proj of a large decode batch (K = dt_rank) goes the same way: its staged 128x128
    // tiles would give only a few workgroups (20 for 256 sequences of a 1280-channel shard)
    if (M <= 64 || (ROLE == kGemmDtProj && AF && M <= 512 && K <= 512)) return few_rows();
    if constexpr (!AF) {
        if (K % 64 == 0 && !(ROLE == kGemmDtProj && K <= 256)) {
            const GemmPlan g = plan_bf16<CF>((GemmRole)ROLE, M, N, K, scratch ? scratch_bytes : 0);
            if (g.tile < 0) return few_rows();
            return dispatch_dma<ROLE, CF>(g, M, N, K, A, lda, B, ldb, C, ldc, s, scratch);
        }
        if (ROLE == kGemmXProj && xproj_decode_skinny(M, N)) return few_rows();
        if constexpr (ROLE == kGemmDtProj) {
            if (dt_few_rows(M, N, K)) return few_rows();
            if (dt_one_round(M, N, K))
                return run_dma<ROLE, 256, 256, 64, 2, 2, 4, CF, true, true>(M, N, K, A, lda, B, ldb, C, ldc, s);
        }
        if (K % 32 == 0) return dispatch_dma32<ROLE, CF>(M, N, K, A, lda, B, ldb, C, ldc, s);
    }
    // staged path: fp32 A (rounded while staging) or a K tail; short K favours more tiles
    const int64_t big_tiles = ((M + 255) / 256) * ((N + 255) / 256);
    if (big_tiles >= 512 && K > 256) return run_bf16<ROLE, 256, 256, 2, 2, AF, CF>(M, N, K, A, lda, B, ldb, C, ldc, s);
    return run_bf16<ROLE, 128, 128, 2, 2, AF, CF>(M, N, K, A, lda, B, ldb, C, ldc, s);
}

}  // namespace

hipError_t launch_round_bf16_rows(const float* a, int64_t lda, void* o, int64_t M, int K, hipStream_t s) {
    const int64_t n8 = M * (K / 8);
    if (n8 <= 0) return hipSuccess;
    SSM_LAUNCH(round_bf16_rows_kernel, dim3((unsigned)((n8 + 255) / 256)), dim3(256), 0, s, a, lda, (bf16*)o, M, K);
    return hipGetLastError();
}

namespace {
size_t f32_splitk_bytes(int64_t M, int64_t N, int64_t K) {
    // float32 operands on 128x128 tiles (more than the 64 rows of the streamed kernel)
    if (M <= 64 || N == 0 || f32_slices(((M + 127) / 128) * ((N + 127) / 128), K) <= 1) return 0;
    const int sp = f32_slices(((M + 63) / 64) * ((N + 63) / 64), K);
    return sp > 1 ? (size_t)sp * M * N * 4 : 0;
}
}  // namespace

int gemm_bf16_slices(GemmRole role, int64_t M, int64_t N, int64_t K, bool c_f32, size_t scratch_bytes) {
    if (M <= 64 || N == 0 || K % 64 != 0 || scratch_bytes == 0) return 1;
    const GemmPlan g = c_f32 ? plan_bf16<true>(role, M, N, K, scratch_bytes) : plan_bf16<false>(role, M, N, K, scratch_bytes);
    return g.tile < 0 ? 1 : g.slices;
}

size_t gemm_splitk_bytes(int64_t M, int64_t N, int64_t K, int a_dt, int b_dt, GemmRole role) {
    if (a_dt == SSM_F32 && b_dt == SSM_F32) {
        const F32Parts g = plan_f32_parts(M, N, K, SIZE_MAX);
        return std::max(f32_splitk_bytes(M, N, K), g.slices > 1 ? (size_t)g.slices * M * N * 4 : 0);
    }
    if (M <= 64 || N == 0 || b_dt != SSM_BF16 || a_dt != SSM_BF16 || K % 64 != 0) return 0;
    if (role == kGemmXProj && M <= 512 && N <= 256) return 0;  // the few-row kernel is about as fast
    // the most that a choice of pick_tile's can use
    int most = 1;
    const int64_t nk = K / 64;
    for (const TileCost& t : kTileCost) {
        const int64_t tiles = ((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn);
        if (!t.split || tiles >= 192) continue;
        for (int d = 2; d <= kMaxSlices && d * kMinSliceK <= nk && tiles * d <= 288; ++d)
            if (nk % d == 0) most = std::max(most, d);
    }
    return most > 1 ? (size_t)most * M * N * 4 : 0;
}

size_t gemm_prefill_scratch(int64_t M, int64_t N, int64_t K, int dt) {
    if (dt == SSM_F32)
        return std::max(f32_splitk_bytes(M, N, K),
                        M <= 64 ? 0 : std::min((size_t)kPartsSlices * M * N * 4, (size_t)kPartsGrid * 256 * 224 * 4));
    return K % 64 == 0 ? splitk_reserve(M, N) : 0;
}

// The decode workspace's K-slice scratch: none where the few-row kernels or the decode tiles
// run unsliced (every batch up to 512 over outputs of 128 of their tiles); else what up to 384
// workgroups of 128x128 tiles would use, which pick_tile may spend on any tile.
size_t gemm_decode_scratch(int64_t M, int64_t N, int64_t K, int dt, GemmRole role) {
    if (dt == SSM_F32) return f32_splitk_bytes(M, N, K);
    if (M <= 64 || N == 0 || K % 64 != 0) return 0;
    if (role == kGemmXProj ? M <= 512 && N <= 256 : decode_tiles(M, N, K)) return 0;
    auto cost = [&](int t, double eff) {
        const int64_t n = ((M + t - 1) / t) * ((N + t - 1) / t);
        return (double)((n + 255) / 256) * t * t / eff;
    };
    int64_t tiles = ((M + 127) / 128) * ((N + 127) / 128);
    if (role == kGemmXProj && N <= 256) tiles = (M + 63) / 64;
    else if (cost(256, 1.0) <= cost(128, 0.83)) return 0;
    if (tiles >= 256) return 0;
    const int64_t nk = K / 64, cap = std::max<int64_t>(1, 384 / tiles);
    int best = 1;
    for (int64_t d = 2; d <= cap && d <= nk / 2; ++d)
        if (nk % d == 0) best = (int)d;
    return best > 1 ? (size_t)best * M * N * 4 : 0;
}

hipError_t launch_gemm_nt(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, int a_dt, const void* B,
                          int64_t ldb, int b_dt, void* C, int64_t ldc, int c_dt, hipStream_t s, GemmRole role,
                          float* scratch, size_t scratch_bytes, bool parts) {
    if (M == 0 || N == 0) return hipSuccess;
    if (b_dt == SSM_F32) {
        // up to 64 rows (a decode step): the weight stream in whole lines
        if (M <= 64) {
            const hipError_t e = launch_gemv_f32_stream(role, M, N, K, (const float*)A, lda, (const float*)B, ldb,
                                                        (float*)C, ldc, s);
            if (e != hipErrorNotSupported) return e;
        }
        auto al16 = [](const void* q) { return ((uintptr_t)q & 15) == 0; };
        if (M <= 8 && K % 4 == 0 && lda % 4 == 0 && ldb % 4 == 0 && al16(A) && al16(B)) {
            const dim3 grid((unsigned)((N + 3) / 4));
#define SSM_F32_GEMV(R)                                                                                              \
    case R:                                                                                                          \
        SSM_LAUNCH(gemv_f32_kernel<R>, grid, dim3(256), 0, s, (int)M, (int)N, (int)K, (const float*)A, lda,         \
                   (const float*)B, ldb, (float*)C, ldc);                                                            \
        break;
            switch (role) {
                SSM_F32_GEMV(kGemmInProj)
                SSM_F32_GEMV(kGemmXProj)
                SSM_F32_GEMV(kGemmDtProj)
                SSM_F32_GEMV(kGemmOutProj)
                default: SSM_F32_GEMV(kGemmGeneric)
            }
#undef SSM_F32_GEMV
            return hipGetLastError();
        }
        // prefill sizes on the DMA tiles (float32 rows moved as bytes, run_dma_f32): when the
        // output has few 128x128 tiles (x_proj: 32), K-slices of 64x64 tiles (4 waves of 32x32,
        // a 4-deep ring of 16 KB stages, two workgroups per CU), whose partials are a quarter of
        // those of 128x128 slices for as many workgroups; else the tile shape of least modelled
        // time (f32_tiles)
        {
            const int64_t tm2 = (M + 127) / 128, tn2 = (N + 127) / 128;
            const bool few = f32_slices(tm2 * tn2, K) > 1;
            const int sp = few ? fit_slices(f32_slices(((M + 63) / 64) * ((N + 63) / 64), K), M, N, scratch_bytes) : 1;
            if (K % kF32BK == 0 && lda % 4 == 0 && ldb % 4 == 0 && al16(A) && al16(B) && al16(C) &&
                256 * lda * 4 < ((int64_t)1 << 31) && 256 * ldb * 4 < ((int64_t)1 << 31)) {
                const float* fA = (const float*)A;
                const float* fB = (const float*)B;
                float* fC = (float*)C;
                // on the bf16 cores when that is faster and no further from float64: its distance
                // is 1.56e-8 sqrt(K / slices) (2-norm, measured on the shapes of gemm_split.h),
                // that of the float32 tiles 1.79e-8 sqrt(K / slices)
                if (parts) {
                    const F32Parts g = plan_f32_parts(M, N, K, scratch ? scratch_bytes : 0);
                    if (sp <= 2 && g.slices * 4 >= sp * 3 && g.us < 0.95f * f32_us(M, N, K, sp)) {
                        float* to = g.slices > 1 ? scratch : fC;
                        const hipError_t e = launch_gemm_f32_parts(g, role, M, N, K, fA, lda, fB, ldb, to,
                                                                   g.slices > 1 ? N : ldc, s);
                        if (e != hipSuccess || g.slices == 1) return e;
                        return reduce_slices_f32(scratch, g.slices, M, N, fC, ldc, s);
                    }
                }
                // (few tiles and a K that does not slice: the register-staged tiles below)
                const F32Tiles t = few ? kF32Tiles64 : f32_tiles(M, N);
                float* part = sp > 1 ? scratch : nullptr;
#define SSM_F32_DMA(R)                                                                                         \
    case R:                                                                                                    \
        switch (t) {                                                                                           \
            case kF32Tiles256: return run_dma_f32<R, 256, 256, 2, 2, 4>(M, N, K, fA, lda, fB, ldb, fC, ldc, s); \
            case kF32Tiles256x224: return run_dma_f32<R, 256, 224, 2, 8, 1>(M, N, K, fA, lda, fB, ldb, fC, ldc, s); \
            case kF32Tiles128x224: return run_dma_f32<R, 128, 224, 2, 4, 2, true>(M, N, K, fA, lda, fB, ldb, fC, ldc, s); \
            case kF32Tiles64: return run_dma_f32<R, 64, 64, 4, 2, 2>(M, N, K, fA, lda, fB, ldb, fC, ldc, s, sp, part); \
            default: return run_dma_f32<R, 128, 128, 2, 2, 4>(M, N, K, fA, lda, fB, ldb, fC, ldc, s); \
        }
                if (few || tm2 * tn2 >= 256) {
                    switch (role) {
                        SSM_F32_DMA(kGemmInProj)
                        SSM_F32_DMA(kGemmXProj)
                        SSM_F32_DMA(kGemmDtProj)
                        SSM_F32_DMA(kGemmOutProj)
                        default: SSM_F32_DMA(kGemmGeneric)
                    }
                }
#undef SSM_F32_DMA
            }
        }
        const int tm = (int)((M + 63) / 64), tn = (int)((N + 63) / 64);
#define SSM_F32_CASE(R)                                                                                             \
    case R:                                                                                                         \
        SSM_LAUNCH(gemm_f32_nt<R>, dim3(tm * tn), dim3(256), 0, s, (int)M, (int)N, (int)K, (const float*)A, \
                           lda, (const float*)B, ldb, (float*)C, ldc, tm, tn);                                      \
        break;
        switch (role) {
            SSM_F32_CASE(kGemmInProj)
            SSM_F32_CASE(kGemmXProj)
            SSM_F32_CASE(kGemmDtProj)
            SSM_F32_CASE(kGemmOutProj)
            default: SSM_F32_CASE(kGemmGeneric)
        }
#undef SSM_F32_CASE
        return hipGetLastError();
    }
    const bool af = a_dt == SSM_F32, cf = c_dt == SSM_F32;
    // the mixer's projections use one operand combination each
    switch (role) {
        case kGemmInProj:
            if (!af && !cf) return dispatch_bf16<kGemmInProj, false, false>(M, N, K, A, lda, B, ldb, C, ldc, s, scratch, scratch_bytes);
            break;
        case kGemmXProj:
            if (!af && cf) return dispatch_bf16<kGemmXProj, false, true>(M, N, K, A, lda, B, ldb, C, ldc, s, scratch, scratch_bytes);
            break;
        case kGemmDtProj:
            if (af && !cf) return dispatch_bf16<kGemmDtProj, true, false>(M, N, K, A, lda, B, ldb, C, ldc, s, scratch, scratch_bytes);
            if (!af && !cf) return dispatch_bf16<kGemmDtProj, false, false>(M, N, K, A, lda, B, ldb, C, ldc, s, scratch, scratch_bytes);
            break;
        case kGemmOutProj:
            if (!af && !cf) return dispatch_bf16<kGemmOutProj, false, false>(M, N, K, A, lda, B, ldb, C, ldc, s, scratch, scratch_bytes);
            break;
        default:
            break;
    }
    if (af && cf) return dispatch_bf16<kGemmGeneric, true, true>(M, N, K, A, lda, B, ldb, C, ldc, s, scratch, scratch_bytes);
    if (af) return dispatch_bf16<kGemmGeneric, true, false>(M, N, K, A, lda, B, ldb, C, ldc, s, scratch, scratch_bytes);
    // bf16 operands: the instances of the projections with this output type
    if (cf) return dispatch_bf16<kGemmXProj, false, true>(M, N, K, A, lda, B, ldb, C, ldc, s, scratch, scratch_bytes);
    return dispatch_bf16<kGemmInProj, false, false>(M, N, K, A, lda, B, ldb, C, ldc, s, scratch, scratch_bytes);
}

}  // namespace ssm
