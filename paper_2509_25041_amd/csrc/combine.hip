// grace_combine: weighted gather of the k expert outputs of every token back to
// token order (the aggregation step after the expert computation, Section 1),
// fp32 accumulation in ascending j, one rounding.
#include "bf16.h"
#include "common.h"

namespace grace {

// Bound by HBM for large batches, by the chain position -> row for small ones: positions and rows of AHEAD
// choices are loaded before the first is used (k = 8, d = 2048, the kernel repeated over six inputs, 1 ahead -> 4: 1 token
// 2.9 -> 2.2 us, 64 tokens 3.9 -> 3.4 us, 512 tokens 7.8 -> 5.3 us; inside a layer step, behind another kernel: 5.6 -> 3.8,
// 6.1 -> 4.6, 7.5 -> 5.4 us).  With AHEAD > 1 an absent row loads row 0, which is not added: a branch around each load
// makes the loads wait for one another (1.3 to 1.5 us more).
template <bool BF16, int AHEAD>
__global__ __launch_bounds__(256) void combine_kernel(const uint4 *__restrict__ y, const int32_t *__restrict__ perm_pos,
                                                      const float *__restrict__ topk_weight, int k, int row_vec,
                                                      int64_t n_rows, const uint4 *__restrict__ y_shared,
                                                      uint4 *__restrict__ out) {
    constexpr int NV = BF16 ? 8 : 4;  // values per 16-byte vector
    const int64_t t = blockIdx.x;
    for (int c = (int)threadIdx.x; c < row_vec; c += 256) {
        float acc[NV];
#pragma unroll
        for (int i = 0; i < NV; ++i) acc[i] = 0.0f;
        uint4 vs = make_uint4(0u, 0u, 0u, 0u);
        if (y_shared) vs = y_shared[t * row_vec + c];
        for (int j0 = 0; j0 < k; j0 += AHEAD) {
            uint4 v[AHEAD];
            float w[AHEAD];
            int32_t p[AHEAD];
            bool row[AHEAD];   // uniform
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) {
                const int64_t a = t * k + min(j0 + i, k - 1);
                p[i] = perm_pos[a];
                w[i] = topk_weight[a];
            }
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) {
                row[i] = j0 + i < k && p[i] >= 0 && p[i] < n_rows;
                if (AHEAD > 1 || row[i]) v[i] = nt_load16(&y[(int64_t)(row[i] ? p[i] : 0) * row_vec + c]);
            }
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) {
                if (!row[i]) continue;
                float f[NV];
                if constexpr (BF16) unpack_bf16x8(v[i], f); else unpack_f32x4(v[i], f);
#pragma unroll
                for (int e = 0; e < NV; ++e) acc[e] = fmaf(w[i], f[e], acc[e]);
            }
        }
        if (y_shared) {
            float f[NV];
            if constexpr (BF16) unpack_bf16x8(vs, f); else unpack_f32x4(vs, f);
#pragma unroll
            for (int i = 0; i < NV; ++i) acc[i] += f[i];
        }
        uint4 o;
        if constexpr (BF16) o = pack_bf16x8(acc); else o = pack_f32x4(acc);
        out[t * row_vec + c] = o;
    }
}

}  // namespace grace

using namespace grace;

// Tokens up to which loading four ahead pays: with 3000 tokens and more the rows in flight of all workgroups are
// enough (3001, 7001, 32768 tokens, k = 6, 8, 6: 18.2 to 19.4, 46.8, 177 us with 1 ahead, 18.2, 45.5, 178 us with 2,
// 19.2, 45.2, 177 us with 4; k = 2, 8192 tokens 31.4 us with 1, 32.3 us with 2).
constexpr int COMBINE_FEW = 1024;

extern "C" int grace_combine(const void *y, const int32_t *perm_pos, const float *topk_weight, int32_t T, int32_t k,
                             int32_t d, grace_dtype dt, const void *y_shared, void *out, void *stream) {
    if (T < 0 || k < 1 || d < 1) return fail(GRACE_EINVAL, "combine: T=%d, k=%d, d=%d invalid", T, k, d);
    if (dt != GRACE_F32 && dt != GRACE_BF16) return fail(GRACE_EINVAL, "combine: unknown dtype %d", (int)dt);
    const size_t el = dt == GRACE_F32 ? 4 : 2;
    if (((size_t)d * el) % 16 != 0) return fail(GRACE_ESHAPE, "combine: row of %zu bytes is not a multiple of 16", (size_t)d * el);
    if ((int64_t)T * k > INT32_MAX) return fail(GRACE_ESHAPE, "combine: T*k exceeds 2^31-1");
    if (T == 0) return GRACE_OK;
    if (!y || !perm_pos || !topk_weight || !out) return fail(GRACE_EINVAL, "combine: null device pointer");
    if ((((uintptr_t)y) | ((uintptr_t)out) | ((uintptr_t)y_shared)) & 15)
        return fail(GRACE_EINVAL, "combine: y, y_shared and out must be 16-byte aligned");
    hipStream_t st = (hipStream_t)stream;
    const int row_vec = (int)((size_t)d * el / 16);
    const int64_t n = (int64_t)T * k;
    auto launch = [&](auto kernel) {
        kernel<<<T, 256, 0, st>>>((const uint4 *)y, perm_pos, topk_weight, k, row_vec, n, (const uint4 *)y_shared, (uint4 *)out);
    };
    const int ahead = (k < 3 ? 2 : 4) >> (T > COMBINE_FEW ? 1 : 0);
    if (dt == GRACE_BF16) launch(ahead == 1 ? combine_kernel<true, 1> : ahead == 2 ? combine_kernel<true, 2> : combine_kernel<true, 4>);
    else launch(ahead == 1 ? combine_kernel<false, 1> : ahead == 2 ? combine_kernel<false, 2> : combine_kernel<false, 4>);
    GRACE_LAUNCH_CHECK("combine_kernel");
    return GRACE_OK;
}
