// Float32 products on the bf16 matrix cores: the tiles of 128 columns.
#include "gemm_split.h"

namespace ssm {
template hipError_t launch_parts_tile<128>(int, int, int64_t, int64_t, int64_t, const float*, int64_t, const float*, int64_t,
                                         float*, int64_t, hipStream_t);
}  // namespace ssm
