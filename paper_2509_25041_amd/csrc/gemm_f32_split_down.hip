// The fp32 split kernels of the down projections.
#include "gemm_f32_split.h"

namespace grace {
namespace split {

const void *down_kernel(int k_groups) {
    return k_groups == 1 ? (const void *)&gemm_f32_split_kernel<false, false, 1> : (const void *)&gemm_f32_split_kernel<false, false, 2>;
}

}  // namespace split
}  // namespace grace
