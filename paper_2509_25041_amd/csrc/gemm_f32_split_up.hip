// The fp32 split kernel of the gate+up projections (a file of its own, as are the two for the down projections: they compile side by side).
#include "gemm_f32_split.h"

namespace grace {
namespace split {

const void *up_kernel() { return (const void *)&gemm_f32_split_kernel<true, false, 1>; }

}  // namespace split
}  // namespace grace
