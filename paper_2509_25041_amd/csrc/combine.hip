// grace_combine: weighted gather of the k expert outputs of every token back to
// token order (the aggregation step after the expert computation, Section 1),
// fp32 accumulation in ascending j, one rounding.
#include "bf16.h"
#include "common.h"
#include "gemm_common.h"

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

// A rank share: rows of y outside [state[4], state[5]) are zero (grace_expert_ffn_up_share / _down_share keep them so)
// and are not read.  A zero row adds w * 0, which is zero or, where the gate weight is not finite, NaN: the sum starts with
// that.  Every wavefront has its token's k positions in its lanes, so a ballot gives the choices to load, taken in ascending
// order, BATCH at a time; a batch's surplus loads have a descriptor without records, read nothing and give zeros, so that
// no branch makes the loads wait for one another.  Bound by HBM (shared rows in, result out) for large batches, by the chain
// position -> row for small ones.  Layer steps in d = 2048, bf16, all rows read -> those of the rank: 32768 tokens, k = 6, 1/22 of the
// rows, shared experts 178 -> 47 us; 7001, k = 8, an eighth 45.4 -> 13.0 us; 3001, k = 6, a seventh, shared experts 18.8 ->
// 6.6 us; d = 4096, 8192 tokens, k = 2, an eighth 31.9 -> 20.4 us.  On a rank that holds every row it takes 0.85 (k = 16) to
// 1.25 (k = 1) of combine_kernel's time; the layer calls that one there.  Batches of 1, 2 and 4: 2048 tokens, k = 8, a quarter of the rows 8.8, 7.3, 7.1 us; k =
// 2, 4096 tokens of 4096 13.6, 12.6, 13.8 us.  Two or four tokens per workgroup gain up to 2.5 us on prefill with few rows and lose
// up to a half for fewer tokens or many rows.  A second pass over the ballots would cost wide rows what they save (a token of d = 4096,
// k = 2, combine_kernel 2.27 us, 256 threads 2.67, 512 threads 2.13; 1000 tokens in fp32 8.4, 9.2, 7.9): rows of more than 256 vectors take
// 512 threads.  Large batches hide the passes behind other tokens, and fewer of them fit a compute unit then (d = 4096, an eighth of the
// rows, 2048 tokens, k = 4 8.3 -> 7.6, 4096 tokens 13.4 -> 14.1, 16384 tokens 37.6 -> 43.8 us).
template <bool BF16, int BATCH, int THREADS>
__global__ __launch_bounds__(THREADS) void combine_share_kernel(const char *__restrict__ y, const int32_t *__restrict__ perm_pos,
                                                            const float *__restrict__ topk_weight, int k, int row_vec,
                                                            int64_t n_rows, const uint4 *__restrict__ y_shared,
                                                            const int32_t *__restrict__ state, uint4 *__restrict__ out) {
    constexpr int NV = BF16 ? 8 : 4;
    const int lane = (int)threadIdx.x & 63;
    const int64_t t = blockIdx.x, a0 = t * k, row_bytes = (int64_t)row_vec * 16;
    const int64_t lo = max(0, state[4]), hi = min(n_rows, (int64_t)state[5]);
    for (int c = (int)threadIdx.x; c - lane < row_vec; c += THREADS) {
        const int cc = min(c, row_vec - 1);   // whole wavefronts stay for the ballots
        int32_t p_lane = perm_pos[a0 + min(lane, k - 1)];
        float w_lane = topk_weight[a0 + min(lane, k - 1)];
        uint4 vs = make_uint4(0u, 0u, 0u, 0u);
        if (y_shared) vs = y_shared[t * row_vec + cc];
        float acc[NV];
#pragma unroll
        for (int e = 0; e < NV; ++e) acc[e] = 0.0f;
        for (int j0 = 0;;) {   // 64 choices at a time
            const bool row = j0 + lane < k && p_lane >= 0 && p_lane < n_rows, here = row && p_lane >= lo && p_lane < hi;
            uint64_t todo = __ballot(here);
            if (__ballot(row && !here && !(w_lane * 0.0f == 0.0f))) {
#pragma unroll
                for (int e = 0; e < NV; ++e) acc[e] = __builtin_nanf("");
            }
            while (todo) {
                u32x4_t v[BATCH];
                float w[BATCH];
#pragma unroll
                for (int b = 0; b < BATCH; ++b) {
                    const int src = todo ? __builtin_ctzll(todo) : 0;
                    const int32_t p = __builtin_amdgcn_readlane(p_lane, src);
                    w[b] = todo ? __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(w_lane), src)) : 0.0f;
                    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void *)(y + (int64_t)p * row_bytes), 0,
                                                                       todo ? (int)row_bytes : 0, 0x00020000);
                    v[b] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, cc * 16, 0, 2 /* nt */);
                    todo &= todo - 1;
                }
#pragma unroll
                for (int b = 0; b < BATCH; ++b) {
                    const uint4 q = make_uint4(v[b][0], v[b][1], v[b][2], v[b][3]);
                    float f[NV];
                    if constexpr (BF16) unpack_bf16x8(q, f); else unpack_f32x4(q, f);
#pragma unroll
                    for (int e = 0; e < NV; ++e) acc[e] = fmaf(w[b], f[e], acc[e]);
                }
            }
            j0 += 64;
            if (j0 >= k) break;
            p_lane = perm_pos[a0 + min(j0 + lane, k - 1)];
            w_lane = topk_weight[a0 + min(j0 + lane, k - 1)];
        }
        if (c >= row_vec) break;
        if (y_shared) {
            float f[NV];
            if constexpr (BF16) unpack_bf16x8(vs, f); else unpack_f32x4(vs, f);
#pragma unroll
            for (int e = 0; e < NV; ++e) acc[e] += f[e];
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
// Tokens up to which combine_share_kernel takes wide rows in one pass.
constexpr int COMBINE_WIDE_MAX = 2048;

static int check_combine_args(const char *who, const void *y, const int32_t *perm_pos, const float *topk_weight, int32_t T,
                              int32_t k, int32_t d, grace_dtype dt, const void *y_shared, const void *out) {
    if (T < 0 || k < 1 || d < 1) return fail(GRACE_EINVAL, "%s: T=%d, k=%d, d=%d invalid", who, T, k, d);
    if (dt != GRACE_F32 && dt != GRACE_BF16) return fail(GRACE_EINVAL, "%s: unknown dtype %d", who, (int)dt);
    const size_t el = dt == GRACE_F32 ? 4 : 2;
    if (((size_t)d * el) % 16 != 0) return fail(GRACE_ESHAPE, "%s: row of %zu bytes is not a multiple of 16", who, (size_t)d * el);
    if ((int64_t)T * k > INT32_MAX) return fail(GRACE_ESHAPE, "%s: T*k exceeds 2^31-1", who);
    if (T == 0) return GRACE_OK;
    if (!y || !perm_pos || !topk_weight || !out) return fail(GRACE_EINVAL, "%s: null device pointer", who);
    if ((((uintptr_t)y) | ((uintptr_t)out) | ((uintptr_t)y_shared)) & 15)
        return fail(GRACE_EINVAL, "%s: y, y_shared and out must be 16-byte aligned", who);
    return GRACE_OK;
}

extern "C" int grace_combine(const void *y, const int32_t *perm_pos, const float *topk_weight, int32_t T, int32_t k,
                             int32_t d, grace_dtype dt, const void *y_shared, void *out, void *stream) {
    const int rc = check_combine_args("combine", y, perm_pos, topk_weight, T, k, d, dt, y_shared, out);
    if (rc != GRACE_OK || T == 0) return rc;
    hipStream_t st = (hipStream_t)stream;
    const int row_vec = (int)((int64_t)d * (dt == GRACE_F32 ? 4 : 2) / 16);
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

extern "C" int grace_combine_share(const void *y, const int32_t *perm_pos, const float *topk_weight, int32_t T, int32_t k,
                                   int32_t d, grace_dtype dt, const void *y_shared, const int32_t *state, void *out,
                                   void *stream) {
    const int rc = check_combine_args("combine_share", y, perm_pos, topk_weight, T, k, d, dt, y_shared, out);
    if (rc != GRACE_OK || T == 0) return rc;
    if (!state) return fail(GRACE_EINVAL, "combine_share: state is null");
    const int64_t row_bytes = (int64_t)d * (dt == GRACE_F32 ? 4 : 2), n = (int64_t)T * k;
    if (row_bytes > INT32_MAX)   // past what a buffer descriptor spans: all rows are read
        return grace_combine(y, perm_pos, topk_weight, T, k, d, dt, y_shared, out, stream);
    auto launch = [&](auto kernel, int threads) {
        kernel<<<T, threads, 0, (hipStream_t)stream>>>((const char *)y, perm_pos, topk_weight, k, (int)(row_bytes / 16), n,
                                                       (const uint4 *)y_shared, state, (uint4 *)out);
    };
    auto by_row = [&](auto narrow, auto wide) { row_bytes <= 256 * 16 || T > COMBINE_WIDE_MAX ? launch(narrow, 256) : launch(wide, 512); };
    if (dt == GRACE_BF16) {
        if (k < 3) by_row(combine_share_kernel<true, 2, 256>, combine_share_kernel<true, 2, 512>);
        else by_row(combine_share_kernel<true, 4, 256>, combine_share_kernel<true, 4, 512>);
    } else {
        if (k < 3) by_row(combine_share_kernel<false, 2, 256>, combine_share_kernel<false, 2, 512>);
        else by_row(combine_share_kernel<false, 4, 256>, combine_share_kernel<false, 4, 512>);
    }
    GRACE_LAUNCH_CHECK("combine_share_kernel");
    return GRACE_OK;
}
