// Down projections of up to 16 tokens (experts' and shared ones) and the combine as one launch.
//
// The combine of a few tokens is a launch of 2 to 4 us that waits for the down projection's.  Here a workgroup owns 8 (or 16) output columns of every
// segment, reads those weight rows of all slots with rows and of the shared experts, and so has all that its columns of the result
// take: no workgroup waits for another.  Its wavefronts deal the segments' parts of K among themselves; partial sums go to LDS, are
// added there in order, rounded as y is, written to y and combined.
//
// Bound by latency, then by the weights: 8 weight rows x 128 bytes per load (whole lines; the lanes of the upper half of the 16 matrix rows
// hold the second 64 bytes, and two matrix instructions, one for each half of K, make sums whose other halves are not looked at), with
// DEPTH steps in flight across the ends of segments.  d = 2048, f = 1024, k = 8: one token, rank with 16 of 64 experts, down and combine 5.4 + 1.9 us in two
// launches -> 7.8 in one, and the launch between them; 16 tokens of 128 experts, f = 768, 8.4 + 3.4 -> 8.6.  Whole steps of one token 16.7 -> 15.4.
// Two shared experts are 2 more segments, not a launch of 5 to 9 us (steps of 2 to 16 tokens 1.15 to 1.35 times as fast).  Where it is the slower one: joins_combine.
#include "ffn_tiny.h"
#include "gemm_stream.h"

namespace grace {

constexpr int DOWN_WAVES = 8, DOWN_THREADS = 64 * DOWN_WAVES;

// Parts of K per segment (their logarithm): enough items for the wavefronts, of two steps or more.
__device__ __forceinline__ int down_parts_log(int segments, int steps) {
    int p = segments <= 4 ? 3 : segments <= 16 ? 2 : segments <= 32 ? 1 : 0;
    while (p > 0 && steps < 2 << p) --p;
    return p;
}

struct DownLds {
    int16_t slot[GRACE_MAX_EXPERTS];               // slots with rows
    int16_t rows[GRACE_MAX_EXPERTS];
    int segments;
};

constexpr int DOWN_FIXED = (sizeof(DownLds) + 15) / 16 * 16;

// EL: bytes per element.  NB: groups of 8 columns.
template <int EL, int NB>
__global__ __launch_bounds__(DOWN_THREADS) void tiny_down_kernel(const TinyDown a) {
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
    static_assert(TINY_DOWN_T * GRACE_MAX_TOPK <= 2 * DOWN_THREADS, "two per thread");
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int i = tid + c * DOWN_THREADS;
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
    const int row_bytes = g.K * EL, steps = (row_bytes + 127) >> 7, parts_log = down_parts_log(segments, steps);
    const int parts = 1 << parts_log, items = segments << parts_log;
    // ---- partial sums
    struct {
        __amdgpu_buffer_rsrc_t a, b;
        uint32_t a_off;
        int item, step, end;
    } ld;   // what is loaded next
    auto begin = [&](int item) {
        ld.item = item;
        if (item >= items) return;
        const int seg = item >> parts_log, p = item & (parts - 1);
        ld.step = (p * steps) >> parts_log;
        ld.end = ((p + 1) * steps) >> parts_log;
        const bool shared = seg >= hit;
        const int slot = __builtin_amdgcn_readfirstlane(shared ? seg - hit : (int)s.slot[shared ? 0 : seg]);
        const int rows = __builtin_amdgcn_readfirstlane(shared ? a.T : (int)s.rows[shared ? 0 : seg]);
        const int64_t lda = shared ? a.shared.lda : g.lda;
        ld.a = rsrc_of(shared ? (const char *)a.shared.A + (int64_t)slot * row_bytes : (const char *)g.A + (int64_t)slot * g.a_slot_rows * g.lda * EL);
        ld.b = rsrc_of((shared ? (const char *)a.shared.B0 + (int64_t)slot * a.shared.kseg_stride * EL : (const char *)g.B0 + (int64_t)slot * g.b_slot_stride * EL) +
                       (int64_t)n0 * row_bytes);
        ld.a_off = (uint32_t)min(r, rows - 1) * (uint32_t)(lda * EL) + (uint32_t)q * 16u;
    };
    uint32_t b_off[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
        b_off[b] = n0 + b * 8 + (r & 7) < g.N ? (uint32_t)(b * 8 + (r & 7)) * (uint32_t)row_bytes + (uint32_t)(r >> 3) * 64u + (uint32_t)q * 16u : NO_DATA;
    u32x4_t rb[DEPTH][NB], ra[DEPTH][2];
    auto load = [&](int p) {
        if (ld.item >= items) return;   // uniform
        const int at = ld.step << 7;
        const bool in0 = at + q * 16 < row_bytes, in1 = at + 64 + q * 16 < row_bytes, in_b = at + (r >> 3) * 64 + q * 16 < row_bytes;
#pragma unroll
        for (int b = 0; b < NB; ++b) rb[p][b] = load16(ld.b, in_b ? b_off[b] : NO_DATA, (uint32_t)at);
        ra[p][0] = load16(ld.a, in0 ? ld.a_off : NO_DATA, (uint32_t)at);
        ra[p][1] = load16(ld.a, in1 ? ld.a_off + 64u : NO_DATA, (uint32_t)at);
        __builtin_amdgcn_sched_barrier(0);
        if (++ld.step == ld.end) begin(ld.item + DOWN_WAVES);
    };
    f32x4_t acc[NB][2];
    auto clear = [&]() {
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[b][0] = acc[b][1] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    };
    auto mma = [&](int p) {
        if constexpr (EL == 2) {
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    acc[b][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, rb[p][b]), __builtin_bit_cast(bf16x8_t, ra[p][h]), acc[b][h], 0, 0, 0);
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v)   // outermost: neighbours do not wait for each other's sums
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        acc[b][h] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(rb[p][b][v]), __uint_as_float(ra[p][h][v]), acc[b][h], 0, 0, 0);
        }
    };
    // element v of lane l: weight row 4 * (l / 16) + v, activation row l % 16; rows 0 to 7 of the first half's sums and 8 to 15 of the second's count
    auto leave = [&](int item) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            f32x4_t sum;
#pragma unroll
            for (int v = 0; v < 4; ++v) sum[v] = acc[b][0][v] + __shfl_xor(acc[b][1][v], 32, 64);
            if (q < 2) *(f32x4_t *)&part[(item * 16 + r) * COLS + b * 8 + 4 * q] = sum;
        }
    };
    begin(wave);
    int item = wave, left = 0;   // in hand
    auto steps_of = [&](int it) { const int p = it & (parts - 1); return (((p + 1) * steps) >> parts_log) - ((p * steps) >> parts_log); };
    if (item < items) left = steps_of(item);
    clear();
#pragma unroll
    for (int p = 0; p < DEPTH; ++p) load(p);
    while (item < items) {
#pragma unroll
        for (int p = 0; p < DEPTH; ++p) {
            if (item >= items) break;
            mma(p);
            load(p);
            if (--left == 0) {
                leave(item);
                clear();
                item += DOWN_WAVES;
                if (item < items) left = steps_of(item);
            }
        }
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const int i = tid + c * DOWN_THREADS, p = c_pos[c];
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
    for (int i = tid; i < (hi0 - lo0) * QUADS; i += DOWN_THREADS) {
        const int row = i / QUADS, quad = i - row * QUADS, col = n0 + quad * 4, at = of[row];
        const f32x4_t y = rounded(sum_of(at >> 4, at & 15, quad));
        *(f32x4_t *)&ylds[i * 4] = y;
        if (col < g.N) store(g.out, lo0 + row, col, y);
    }
    __syncthreads();
    for (int i = tid; i < a.T * QUADS; i += DOWN_THREADS) {
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
static int items_most(int S, int n_shared) { return std::max(64, S + n_shared); }   // down_parts_log leaves 64 or one per segment
int tiny_down_lds(int T, int k, int S, int n_shared, int N, int n_cu) {
    const int n = T * k, cols = 8 * down_groups(N, n_cu);
    return DOWN_FIXED + (n + 7) / 8 * 16 + (n + 1) / 2 * 16 + (items_most(S, n_shared) * 16 + n) * cols * 4;
}
int tiny_down_blocks(int N, int n_cu) { return (N + 8 * down_groups(N, n_cu) - 1) / (8 * down_groups(N, n_cu)); }
const void *tiny_down_kernel_of(grace_dtype dt, int N, int n_cu) {
    const bool wide = down_groups(N, n_cu) == 2;
    if (dt == GRACE_BF16) return wide ? (const void *)tiny_down_kernel<2, 2> : (const void *)tiny_down_kernel<2, 1>;
    return wide ? (const void *)tiny_down_kernel<4, 2> : (const void *)tiny_down_kernel<4, 1>;
}
void launch_tiny_down(const TinyDown &a, grace_dtype dt, int lds, int n_cu, hipStream_t st) {
    TinyDown args = a;
    args.items_most = items_most(a.experts.S, a.n_shared);
    void *params[] = {&args};
    (void)hipLaunchKernel(tiny_down_kernel_of(dt, a.experts.N, n_cu), dim3((unsigned)tiny_down_blocks(a.experts.N, n_cu)), dim3(DOWN_THREADS), params, lds, st);
}

}  // namespace grace
