// The fp32 split kernels of the shared experts' down projection, whose weights' K axis is cut in segments.
#include "gemm_f32_split.h"

namespace grace {
namespace split {

const void *shared_down_kernel(int k_groups) {
    return k_groups == 1 ? (const void *)&gemm_f32_split_kernel<false, true, 1> : (const void *)&gemm_f32_split_kernel<false, true, 2>;
}

}  // namespace split
}  // namespace grace
