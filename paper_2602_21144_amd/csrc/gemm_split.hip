// Float32 products on the bf16 matrix cores (gemm_split.h): the choice of the tile and of K-slices.
#include <algorithm>

#include "gemm_tiles.h"

namespace ssm {

// instantiated in gemm_split_<BN>.hip
template <int BN>
hipError_t launch_parts_tile(int role, int slices, int64_t M, int64_t N, int64_t K, const float* A, int64_t lda,
                             const float* B, int64_t ldb, float* C, int64_t ldc, hipStream_t s);

namespace {

// The tiles' prices, as those of the bf16 table (gemm.hip): launch + rounds x (a x stages + b), a
// rising with the share of the CUs that are busy (the clock falls under MFMA load). Fitted over 968
// runs on 110 shapes, M = 74 .. 28377, N = 80 .. 14336, K = 64 .. 8192 (median error 2%); the
// cheapest is within 1% of the best for 9 shapes in 10 and within 8% for all.
struct PartsCost {
    int bn;
    float a, fill, b;
};
constexpr PartsCost kPartsCost[] = {
    {224, 3.05f, 0.59f, 15.7f}, {192, 2.74f, 0.45f, 11.8f}, {160, 2.36f, 0.38f, 10.2f}, {128, 2.09f, 0.34f, 7.6f}};

float parts_us(const PartsCost& t, int64_t wg, float nk) {
    const float r = wg <= 4 * 256 ? (float)((wg + 255) / 256) : (float)wg / 256.0f + 0.6f;
    return 2.0f + r * ((t.a + t.fill * (float)std::min<int64_t>(wg, 256) / 256.0f) * nk + t.b);
}

}  // namespace

F32Parts plan_f32_parts(int64_t M, int64_t N, int64_t K, size_t scratch_bytes) {
    F32Parts best{128, 1, 1e30f};
    if (M <= 64 || K % kSplitBK != 0) return best;
    const int64_t nk = K / kSplitBK;
    for (const PartsCost& t : kPartsCost) {
        const int64_t tiles = ((M + 255) / 256) * ((N + t.bn - 1) / t.bn);
        for (int d = 1; d <= kPartsSlices; ++d) {
            const size_t bytes = (size_t)d * M * N * 4;
            if (d > 1 && (tiles * d > kPartsGrid || nk / d < 4 || bytes > scratch_bytes)) break;
            if (nk % d != 0) continue;
            const float us = parts_us(t, tiles * d, (float)(nk / d)) + (d > 1 ? split_reduce_us(bytes) : 0.0f);
            if (us < best.us) best = F32Parts{t.bn, d, us};
        }
    }
    return best;
}

hipError_t launch_gemm_f32_parts(const F32Parts& p, int role, int64_t M, int64_t N, int64_t K, const float* A, int64_t lda,
                                 const float* B, int64_t ldb, float* C, int64_t ldc, hipStream_t s) {
    switch (p.bn) {
        case 224: return launch_parts_tile<224>(role, p.slices, M, N, K, A, lda, B, ldb, C, ldc, s);
        case 192: return launch_parts_tile<192>(role, p.slices, M, N, K, A, lda, B, ldb, C, ldc, s);
        case 160: return launch_parts_tile<160>(role, p.slices, M, N, K, A, lda, B, ldb, C, ldc, s);
        default: return launch_parts_tile<128>(role, p.slices, M, N, K, A, lda, B, ldb, C, ldc, s);
    }
}

}  // namespace ssm
