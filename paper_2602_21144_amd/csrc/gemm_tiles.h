// Helpers of the DMA-fed GEMM kernels (gemm.hip, gemm_split.h).
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

// Float32 products on the bf16 matrix cores (gemm_split.h). The plan is the cheapest tile and
// number of K-slices whose partials fit the scratch (us: its price, 1e30 where it does not apply);
// the product leaves slice k's sums in C + k M ldc.
constexpr int kSplitBK = 32;  // k per stage: one 128-byte line of every row
constexpr int kPartsSlices = 8, kPartsGrid = 288;  // K-slices: at most 8, over grids of up to 288 workgroups
struct F32Parts {
    int bn, slices;
    float us;
};
F32Parts plan_f32_parts(int64_t M, int64_t N, int64_t K, size_t scratch_bytes);
hipError_t launch_gemm_f32_parts(const F32Parts& p, int role, int64_t M, int64_t N, int64_t K, const float* A, int64_t lda,
                                 const float* B, int64_t ldb, float* C, int64_t ldc, hipStream_t s);

// us of the pass that adds K-slices: float32 partials written and read again (fitted on the bf16
// products' shapes)
inline float split_reduce_us(size_t bytes) { return 3.8f + 0.36f * (float)bytes * 1e-6f; }

}  // namespace ssm
