// Down projections of up to 16 tokens (experts' and shared ones) and the combine as one launch.
//
// The combine of a few tokens is a launch of 2 to 4 us that waits for the down projection's.  Here a workgroup owns 8 (or 16) output columns of every
// segment, reads those weight rows of all slots with rows and of the shared experts, and so has all that its columns of the result
// take: no workgroup waits for another.  Its wavefronts deal the segments' parts of K among themselves; partial sums go to LDS, are
// added there in order, rounded as y is, written to y and combined.
//
// Bound by latency, then by the weights: 8 weight rows x 128 bytes per load (whole lines; tiny_parts.h).  d = 2048, f = 1024, k = 8: one token, rank with 16 of 64 experts, down and combine 5.4 + 1.9 us in two
// launches -> 7.5 in one, and the launch between them; 16 tokens of 128 experts, f = 768, 8.4 + 3.4 -> 8.6.  Whole steps of one token 16.7 -> 15.4.
// Two shared experts are 2 more segments, not a launch of 5 to 9 us (steps of 2 to 16 tokens 1.15 to 1.35 times as fast).  Where it is the slower one: joins_combine.
#include "ffn_tiny.h"
#include "gemm_stream.h"
#include "tiny_parts.h"

namespace grace {

struct DownLds {
    int16_t slot[GRACE_MAX_EXPERTS];               // slots with rows
    int16_t rows[GRACE_MAX_EXPERTS];
    int segments;
};

constexpr int DOWN_FIXED = (sizeof(DownLds) + 15) / 16 * 16;

// EL: bytes per element.  NB: groups of 8 columns.  OCTETS: up to 8 tokens (a kernel of its own: with both walks in one that of up to 8 is 0.4 us slower).
template <int EL, int NB, bool OCTETS>
__global__ __launch_bounds__(PART_THREADS) void tiny_down_kernel(const TinyDown a) {
    constexpr int DEPTH = NB == 1 ? 6 : 4, COLS = 8 * NB;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    DownLds &s = *(DownLds *)smem;
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), r = lane & 15, q = lane >> 4;
    const int n0 = (int)blockIdx.x * COLS, n = a.T * a.k;
    // of each of the rank's rows: segment * 16 + row in it; of each choice: its row of the rank (-1: another's, -2: another's with a weight that is
    // not finite) and weight; partial sums [item][16 rows][COLS]; y, rounded, [row][COLS]
    int16_t *const of = (int16_t *)(smem + DOWN_FIXED);
    float2 *const choice = (float2 *)(of + (n + 7) / 8 * 8);
    float *const part = (float *)(choice + (n + 1) / 2 * 2);
    float *const ylds = part + a.items_most * 16 * COLS;
    const GemmArgs &g = a.experts;
    const StaleRows stale = stale_rows(g);
    // ---- segments with rows, the tokens' choices (up to two per thread wait in registers)
    int c_pos[2];
    float c_weight[2];
    static_assert(TINY_DOWN_T * GRACE_MAX_TOPK <= 2 * PART_THREADS, "two per thread");
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int i = tid + c * PART_THREADS;
        c_pos[c] = i < n ? a.perm_pos[i] : -1;
        c_weight[c] = i < n ? a.weight[i] : 0.0f;
    }
    const int lo0 = max(0, min(n, __builtin_amdgcn_readfirstlane(g.seg_off[0]))), hi0 = max(lo0, min(n, __builtin_amdgcn_readfirstlane(g.seg_off[g.S])));
    if (wave == 0) {
        int count = 0;
        for (int s0 = 0; s0 < g.S; s0 += 64) {
            const int slot = s0 + lane, lo = slot < g.S ? g.seg_off[slot] : 0, rows = slot < g.S ? min(g.seg_off[slot + 1] - lo, TINY_DOWN_T) : 0;
            const uint64_t hit = __ballot(rows > 0);
            const int at = count + (int)__popcll(hit & lanemask_lt());
            if (rows > 0) {
                s.slot[at] = (int16_t)slot;
                s.rows[at] = (int16_t)rows;
                for (int i = 0; i < rows; ++i)
                    if (lo - lo0 + i >= 0 && lo - lo0 + i < n) of[lo - lo0 + i] = (int16_t)(at * 16 + i);
            }
            count += (int)__popcll(hit);
        }
        if (lane == 0) s.segments = count;
    }
    __syncthreads();
    const int hit = __builtin_amdgcn_readfirstlane(s.segments), segments = hit + a.n_shared;
    const int row_bytes = g.K * EL, steps = (row_bytes + 127) >> 7, parts_log = parts_log_of(segments, steps), parts = 1 << parts_log, items = segments << parts_log;
    // ---- partial sums
    uint32_t b_off[NB], a_off = 0;
#pragma unroll
    for (int b = 0; b < NB; ++b)
        b_off[b] = n0 + b * 8 + (r & 7) < g.N ? (uint32_t)(b * 8 + (r & 7)) * (uint32_t)row_bytes + (uint32_t)(r >> 3) * 64u + (uint32_t)q * 16u : NO_DATA;
    __amdgpu_buffer_rsrc_t a_rsrc, b_rsrc;
    walk_parts<EL, NB, DEPTH, OCTETS>(
        wave, items, parts_log, steps,
        [&](int seg) {
            const bool shared = seg >= hit;
            const int slot = __builtin_amdgcn_readfirstlane(shared ? seg - hit : (int)s.slot[shared ? 0 : seg]);
            const int rows = __builtin_amdgcn_readfirstlane(shared ? a.T : (int)s.rows[shared ? 0 : seg]);
            const int64_t lda = shared ? a.shared.lda : g.lda;
            a_rsrc = rsrc_of(shared ? (const char *)a.shared.A + (int64_t)slot * row_bytes : (const char *)g.A + (int64_t)slot * g.a_slot_rows * g.lda * EL);
            b_rsrc = rsrc_of((shared ? (const char *)a.shared.B0 + (int64_t)slot * a.shared.kseg_stride * EL : (const char *)g.B0 + (int64_t)slot * g.b_slot_stride * EL) +
                             (int64_t)n0 * row_bytes);
            a_off = (uint32_t)min(OCTETS ? r & 7 : r, rows - 1) * (uint32_t)(lda * EL) + (OCTETS ? (uint32_t)(r >> 3) * 64u : 0u) + (uint32_t)q * 16u;
        },
        [&](int at, u32x4_t (&rb)[NB], u32x4_t (&ra)[OCTETS ? 1 : 2]) {
            const bool in = at + (r >> 3) * 64 + q * 16 < row_bytes;
#pragma unroll
            for (int b = 0; b < NB; ++b) rb[b] = load16(b_rsrc, in ? b_off[b] : NO_DATA, (uint32_t)at);
            if constexpr (OCTETS) {
                ra[0] = load16(a_rsrc, in ? a_off : NO_DATA, (uint32_t)at);
            } else {
                ra[0] = load16(a_rsrc, at + q * 16 < row_bytes ? a_off : NO_DATA, (uint32_t)at);
                ra[1] = load16(a_rsrc, at + 64 + q * 16 < row_bytes ? a_off + 64u : NO_DATA, (uint32_t)at);
            }
        },
        [&](int item, int b, const f32x4_t &sum) {
            if (q < 2 && (!OCTETS || r < 8)) *(f32x4_t *)&part[(item * 16 + r) * COLS + b * 8 + 4 * q] = sum;
        });
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int i = tid + c * PART_THREADS, p = c_pos[c];
        const bool here = p >= lo0 && p < hi0, row = p >= 0 && p < n;
        if (i < n) choice[i] = make_float2(__int_as_float(here ? p - lo0 : row && !(c_weight[c] * 0.0f == 0.0f) ? -2 : -1), c_weight[c]);
    }
    __syncthreads();
    // ---- y, then the combine: four columns per thread
    constexpr int QUADS = COLS / 4;
    auto sum_of = [&](int seg, int row, int quad) {   // in the order of the parts
        const float *at = &part[((seg << parts_log) * 16 + row) * COLS + quad * 4];
        f32x4_t sum = *(const f32x4_t *)at;
        for (int p = 1; p < parts; ++p) sum += *(const f32x4_t *)(at + p * 16 * COLS);
        return sum;
    };
    auto rounded = [&](f32x4_t v) {
        if constexpr (EL == 2) {
            const uint32_t x = pack_bf16x2(v[0], v[1]), y = pack_bf16x2(v[2], v[3]);
            v = f32x4_t{bf16_lo_to_f32(x), bf16_hi_to_f32(x), bf16_lo_to_f32(y), bf16_hi_to_f32(y)};
        }
        return v;
    };
    auto store = [&](void *base, int64_t row, int col, f32x4_t v) {
        if constexpr (EL == 2) *(uint2 *)((uint16_t *)base + row * g.N + col) = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
        else *(float4 *)((float *)base + row * g.N + col) = make_float4(v[0], v[1], v[2], v[3]);
    };
    for (int i = tid; i < (hi0 - lo0) * QUADS; i += PART_THREADS) {
        const int row = i / QUADS, quad = i - row * QUADS, col = n0 + quad * 4, at = of[row];
        const f32x4_t y = rounded(sum_of(at >> 4, at & 15, quad));
        *(f32x4_t *)&ylds[i * 4] = y;
        if (col < g.N) store(g.out, lo0 + row, col, y);
    }
    __syncthreads();
    for (int i = tid; i < a.T * QUADS; i += PART_THREADS) {
        const int t = i / QUADS, quad = i - t * QUADS, col = n0 + quad * 4;
        if (col >= g.N) continue;
        f32x4_t out = {0.0f, 0.0f, 0.0f, 0.0f}, ys = out;
        bool nan = false;   // a zero row of another rank adds w * 0
        if (a.n_shared) {
            ys = sum_of(hit, t, quad);
            for (int e = 1; e < a.n_shared; ++e) ys += sum_of(hit + e, t, quad);
            ys = rounded(ys);
            store(a.shared.out, t, col, ys);
        }
        for (int j0 = 0; j0 < a.k; j0 += 4) {   // four choices' reads at a time
            f32x4_t y[4];
            float w[4];
            int row[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float2 c = choice[t * a.k + min(j0 + j, a.k - 1)];
                row[j] = j0 + j < a.k ? __float_as_int(c.x) : -1;
                w[j] = c.y;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) y[j] = *(const f32x4_t *)&ylds[(max(row[j], 0) * QUADS + quad) * 4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                nan |= row[j] == -2;
                if (row[j] < 0) continue;
#pragma unroll
                for (int v = 0; v < 4; ++v) out[v] = fmaf(w[j], y[j][v], out[v]);
            }
        }
        if (nan) out = f32x4_t{__builtin_nanf(""), __builtin_nanf(""), __builtin_nanf(""), __builtin_nanf("")};
        if (a.n_shared) out += ys;
        store(a.out, t, col, out);
    }
    clear_stale_rows(g, stale);
}

static int down_groups(int N, int n_cu) { return (N + 7) / 8 > n_cu + n_cu / 2 ? 2 : 1; }
int tiny_down_lds(int T, int k, int S, int n_shared, int N, int n_cu) {
    const int n = T * k, cols = 8 * down_groups(N, n_cu);
    return DOWN_FIXED + (n + 7) / 8 * 16 + (n + 1) / 2 * 16 + (parts_most(S, n_shared) * 16 + n) * cols * 4;
}
int tiny_down_blocks(int N, int n_cu) { return (N + 8 * down_groups(N, n_cu) - 1) / (8 * down_groups(N, n_cu)); }
template <int EL, int NB>
static const void *kernel_of(int T) {
    return T <= 8 ? (const void *)tiny_down_kernel<EL, NB, true> : (const void *)tiny_down_kernel<EL, NB, false>;
}
const void *tiny_down_kernel_of(grace_dtype dt, int T, int N, int n_cu) {
    const bool wide = down_groups(N, n_cu) == 2;
    if (dt == GRACE_BF16) return wide ? kernel_of<2, 2>(T) : kernel_of<2, 1>(T);
    return wide ? kernel_of<4, 2>(T) : kernel_of<4, 1>(T);
}
void launch_tiny_down(const TinyDown &a, grace_dtype dt, int lds, int n_cu, hipStream_t st) {
    TinyDown args = a;
    args.items_most = parts_most(a.experts.S, a.n_shared);
    void *params[] = {&args};
    (void)hipLaunchKernel(tiny_down_kernel_of(dt, a.T, a.experts.N, n_cu), dim3((unsigned)tiny_down_blocks(a.experts.N, n_cu)), dim3(PART_THREADS), params, lds, st);
}

}  // namespace grace
