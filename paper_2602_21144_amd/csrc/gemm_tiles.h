// Helpers of the DMA-fed GEMM kernels (gemm.hip, gemm_split.hip).
#pragma once
#include <utility>

#include "common.h"

namespace ssm {
namespace {

// Map the linear workgroup id to an output tile. Workgroups are dispatched round robin
// over the 8 XCDs; regroup so each XCD gets a contiguous run of tiles, and order the
// tiles in groups of 4 tile-rows so that a run shares A panels and B panels in its L2
// (groups of 4 took dt_proj's 2560 short tiles from 31 to 28 us; 8 and 16 measured the
// same or slower on every projection).
__device__ __forceinline__ void tile_of(int tiles_m, int tiles_n, int& tm, int& tn) {
    int nwg = gridDim.x;
    int bid = blockIdx.x;
    if ((nwg & 7) == 0) bid = (bid & 7) * (nwg >> 3) + (bid >> 3);
    constexpr int G = 4;
    int per_group = G * tiles_n;
    int grp = bid / per_group;
    int first = grp * G;
    int gm = min(tiles_m - first, G);
    int r = bid - grp * per_group;
    tm = first + r % gm;
    tn = r / gm;
}

// f(integral_constant<int, i>) for i = 0 .. N-1, unrolled at compile time
template <typename F, int... I>
__device__ __forceinline__ void static_for_seq(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F> __device__ __forceinline__ void static_for(F&& f) {
    static_for_seq(f, std::make_integer_sequence<int, N>{});
}

// chunk permutation of an LDS row: 16 lanes reading one chunk column of 16 consecutive
// rows hit distinct 16-byte bank groups (128-byte rows: key (r>>1)&7; 64-byte: (r>>2)&3)
template <int BK> __device__ __forceinline__ int swz_k(int row, int chunk) {
    if constexpr (BK == 64) return chunk ^ ((row >> 1) & 7);
    else return chunk ^ ((row >> 2) & 3);
}

}  // namespace

// Split float32 operands (gemm_split.hip): the rows of A and B as f16 halves [K / 32][hi 32 |
// lo 32] and a power of two per row; kSplitBad marks a row that the split does not suit.
constexpr int kSplitBad = -(1 << 28);
constexpr float kSplitSmall = 0.25f;  // below it (rows scaled to 2^15) lo may not be a normal f16
// nonzero values of a row that may lie below it: of normally distributed rows, far fewer do
__host__ __device__ inline int split_small_limit(int K) { return 4 + K / 64; }
constexpr int64_t kSplitMaxK = 8192;  // a row is held in the registers of one workgroup
struct SplitOperands {
    void *a, *b;       // [M][2K], [N][2K] f16
    int32_t *ea, *eb;  // [M], [N]
};
// bytes of halves that such a product needs (monotone in M; 0: it is not run this way), its
// modelled time, and the product itself: every output but those of marked rows and columns.
// The caller launches the float32 tiles behind it on the exponents it returns.
float gemm_f32_split_us(int64_t M, int64_t N, int64_t K);
hipError_t launch_gemm_f32_split(int role, int64_t M, int64_t N, int64_t K, const float* A, int64_t lda, const float* B,
                                 int64_t ldb, float* C, int64_t ldc, void* halves, hipStream_t s, SplitOperands* out);

}  // namespace ssm
