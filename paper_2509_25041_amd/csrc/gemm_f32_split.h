// fp32 grouped GEMM on the bf16 matrix cores, for batches of more than 64 tokens: every fp32 value is split into three bf16 values whose
// sum it is, and a product is the sum of the six partial products down to 2^-18 of it.
//
// x = x1 + x2 + x3 exactly, each part x's next 8 bits (rounded to nearest, so the parts have signs of their own); a product a b is
// a1 b1 + (a1 b2 + a2 b1) + (a1 b3 + a2 b2 + a3 b1), each of them exact in fp32.  What is left out, a2 b3 + a3 b2 + a3 b3, is 2^-27.5 of the
// product (root mean square; the rounding of one fp32 product 2^-25.2), 0.85 * 2^-24 at most.  The leading products have accumulators of
// their own, so what an addition rounds away is a part of their sum once per 32 K, and of the others 2^-8 of that.  Error of expert FFNs
// against 64 bits (2-norm; the fp32 matrix instruction with its chains of K / 16 -> this kernel): d = 1024, f = 2816 6.4e-7 -> 3.8e-7, d =
// 2048, f = 768 6.5e-7 -> 4.5e-7, d = 548, f = 1388 4.6e-7 -> 3.9e-7.  Of a sum with a single product other than zero, 2^-24: 0.424 -> 0.433
// (root mean square), 1.0 -> 1.6 at most.
//
// Values below 2^-110 lose their third part and products can leave the range of fp32 on the way that their sum stays in, so every sum is
// looked at when it is done: one that is not far above all that can have got lost, or not finite, is computed again with the fp32
// instruction (doubtful, by_f32: about 1e-26 with rows of ordinary size).  It is each element's own matter, and the order in which a sum is
// taken depends on its weights and the host's sizes alone: a row's result does not depend on the batch around it.
//
// Bound by what the fp32 instruction is not: six bf16 instructions of 16 cycles take 96 for what takes that one 256, so what is left
// is the split, the LDS and above all the operands' way to the compute units (a tile of 80 x 128 has 25 operations per byte).
// Hence: values are split once, on their way to LDS (three planes, 1.5 times the bytes), between the matrix instructions of the step before
// (multiplied first and split then 114 instead of 100 us below); a step's loads are issued as soon as the registers they land in have been
// split, so they have AHEAD whole steps; two weight fragments per wavefront share each activation fragment's read where there
// are tiles enough.  80 rows: two groups of four wavefronts fill the LDS.
// Where a launch's tiles are few, K long (down projections), the two groups of a compute unit share a tile, each with half of K (d =
// 1024, f = 2816, 989 rows in 9 segments 84 -> 68 us, 332 rows 46 -> 39, 114 rows 46 -> 35; where: split_groups in ffn.hip).
//
// d = 1024, f = 2816, cold weights, fp32 instruction (96 x 64 tiles, or streamed) -> this kernel, us: 989 rows in 9 segments, gate+up 135 ->
// 103, down 101 -> 68; 332 rows 78 -> 55, 63 -> 39; 2000 rows in 16 segments 260 -> 181, 160 -> 132; 16000 rows 1725 -> 1140 (162
// TFLOP/s, the fp32 instruction's own peak is 157), 840 -> 570.  66 rows, bound by the weights (207 MB), 43 -> 47.
#pragma once
#include <type_traits>
#include <utility>

#include "bf16.h"
#include "gemm_bf16_mid.h"

namespace grace {
namespace split {

constexpr int BM = 80, BK = 32;   // a step is one 128-byte line of fp32 per row
constexpr int MAX_MF = BM / 16, B_WAVE_ROWS = 32;
constexpr int A_PLANE = BM * BK * 2, B_PLANE = B_WAVE_ROWS * BK * 2;
constexpr int BUFFER_BYTES = 3 * (A_PLANE + 4 * B_PLANE), GROUP_BYTES = 2 * BUFFER_BYTES;   // LDS of four wavefronts
static_assert(2 * GROUP_BYTES <= 160 * 1024, "two groups per compute unit");

// The products that make one, the smallest first: part of the weight, part of the activation (0: the leading ones).
constexpr int PRODUCTS = 6, PART_B[] = {2, 1, 0, 1, 0, 0}, PART_A[] = {0, 1, 2, 0, 1, 0};

// f(0) .. f(N - 1) with the numbers as types: the order of the instructions and which register each uses are set here, not by unrolling
template <typename F, int... I>
__device__ __forceinline__ void each_of(F &&f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void each(F &&f) {
    each_of(f, std::make_integer_sequence<int, N>{});
}

// Can underflow or overflow have touched a sum of K products, as the parts give it?  am, bm: the largest magnitudes of its two rows.  What can
// get lost on the way, parts, partial products and sums below 2^-126, is less than K * 2^-125 * (am + bm + 8); a sum of 2^25 times that
// does not feel it.
__device__ __forceinline__ float least_of(float am, float bm, int K) { return (float)K * 0x1p-100f * (am + bm + 8.0f); }
__device__ __forceinline__ bool doubtful(float sum, float am, float bm, int K) {
    const float s = fabsf(sum);
    if (s >= least_of(am, bm, K) && s < INFINITY) return false;
    if (s == 0.0f && (am == 0.0f || bm == 0.0f)) return false;
    return !(s != s && am < 0x1p47f && bm < 0x1p47f);   // no product overflows: it is the NaN of an operand
}
// the kernels, each compiled in a .hip file of its own (shared_down: weights' K axis in segments)
const void *up_kernel();
const void *down_kernel(int k_groups);
const void *shared_down_kernel(int k_groups);

template <bool FUSED_UP>
struct Shape {
    static constexpr int BN = FUSED_UP ? 64 : 128;    // output columns of a whole tile
};

typedef __attribute__((ext_vector_type(2))) uint32_t u32x2_t;

// bytes from a plane's start: two rows of 64 bytes per 128-byte line, the 16-byte chunks of a line permuted (no bank conflicts)
__device__ __forceinline__ int chunk_at(int row, int c) {
    const int line = row >> 1;
    return line * 128 + ((((row & 1) * 4 + c) ^ (line & 7)) * 16);
}

// x = hi + mid + lo, each rounded to bf16: the remainders are exact, and 24 bits fit three times 8.
__device__ __forceinline__ void split2(float x, float y, uint32_t &hi, uint32_t &mid, uint32_t &lo) {
    hi = pack_bf16x2(x, y);
    x -= bf16_lo_to_f32(hi);
    y -= bf16_hi_to_f32(hi);
    mid = pack_bf16x2(x, y);
    x -= bf16_lo_to_f32(mid);
    y -= bf16_hi_to_f32(mid);
    lo = pack_bf16x2(x, y);
}

// What a tile leaves in LDS for the check of its sums: the largest magnitudes of its rows, and the sums of a tile that did not pass at once.
template <int K_GROUPS>
struct Left {
    alignas(16) float a_most[K_GROUPS][BM];
    alignas(16) float b_most[K_GROUPS][4][B_WAVE_ROWS];
    f32x4_t sums[4][MAX_MF * 2][64];   // [wavefront][fragment][lane]
    __device__ __forceinline__ float a(int row) const { return K_GROUPS > 1 ? fmaxf(a_most[0][row], a_most[K_GROUPS - 1][row]) : a_most[0][row]; }
    __device__ __forceinline__ float b4(int wave, int row) const {   // of four rows, the first a multiple of 4
        f32x4_t m = *(const f32x4_t *)&b_most[0][wave][row];
        float most = fmaxf(fmaxf(m[0], m[1]), fmaxf(m[2], m[3]));
        if (K_GROUPS > 1) {
            m = *(const f32x4_t *)&b_most[K_GROUPS - 1][wave][row];
            most = fmaxf(most, fmaxf(fmaxf(m[0], m[1]), fmaxf(m[2], m[3])));
        }
        return most;
    }
    __device__ __forceinline__ float b(int wave, int row) const {
        return K_GROUPS > 1 ? fmaxf(b_most[0][wave][row], b_most[K_GROUPS - 1][wave][row]) : b_most[0][wave][row];
    }
};
static_assert(sizeof(Left<2>) <= GROUP_BYTES, "one group's LDS holds it");

// Operands of a wavefront's part of a tile straight from memory.  Two fragments of weights: gate and up, or the wavefront's two (wn: its
// first output column; nj: how many it has).
template <bool FUSED_UP>
struct FromMemory {
    __amdgpu_buffer_rsrc_t a, b[2];
    uint32_t b_off[2];
    __device__ __forceinline__ FromMemory(const GemmArgs &g, int slot, int m0, int wn, int nj, int r) {
        const int64_t b_first = ((int64_t)slot * g.b_slot_stride + (int64_t)wn * g.ldb) * 4;
        a = rsrc_of((const char *)g.A + (int64_t)m0 * g.lda * 4);
        b[0] = rsrc_of((const char *)g.B0 + b_first);
        b[1] = rsrc_of((FUSED_UP ? (const char *)g.B1 : (const char *)g.B0) + b_first);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int n = FUSED_UP ? r : j * 16 + r;
            b_off[j] = wn + n < g.N && (FUSED_UP || j < nj) ? (uint32_t)n * (uint32_t)(g.ldb * 4) : NO_DATA;
        }
    }
};
// COUNT times 16 rows from row `first` on (of the tile) with the fp32 matrix instruction; the sums whose bits are set go out.
template <bool FUSED_UP, bool SEG_K, int COUNT>
__device__ __forceinline__ void rows_by_f32(const GemmArgs &g, const FromMemory<FUSED_UP> &from, int m0, int m_end, int first, int wn, int lane, uint64_t again) {
    const int r = lane & 15, q = lane >> 4;
    uint32_t a_off[COUNT];
    f32x4_t part[COUNT][2][4];   // chains of K / 16 additions
#pragma unroll
    for (int i = 0; i < COUNT; ++i) {
        const int row = first + i * 16 + r;
        a_off[i] = m0 + row < m_end ? (uint32_t)row * (uint32_t)(g.lda * 4) : NO_DATA;
#pragma unroll
        for (int v = 0; v < 4; ++v) part[i][0][v] = part[i][1][v] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    }
    constexpr int UNROLL = COUNT == 1 ? 8 : 1;
#pragma unroll UNROLL
    for (int k0 = 0; k0 < g.K; k0 += 16) {
        const int k = k0 + 4 * q;   // (K is a multiple of 4)
        const uint32_t ka = k < g.K ? (uint32_t)k * 4u : NO_DATA;
        const uint32_t kb = SEG_K && k < g.K ? (uint32_t)(koff(g, k) * 4) : ka;
        f32x4_t fb[2], fa[COUNT];
#pragma unroll
        for (int j = 0; j < 2; ++j) fb[j] = __builtin_bit_cast(f32x4_t, load16(from.b[j], offset_with(from.b_off[j], kb), 0));
#pragma unroll
        for (int i = 0; i < COUNT; ++i) fa[i] = __builtin_bit_cast(f32x4_t, load16(from.a, offset_with(a_off[i], ka), 0));
#pragma unroll
        for (int i = 0; i < COUNT; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int j = 0; j < 2; ++j) part[i][j][v] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[j][v], fa[i][v], part[i][j][v], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < COUNT; ++i) {
        float *const o = (float *)g.out + (int64_t)(m0 + first + i * 16 + r) * g.ldo + wn + 4 * q;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float h = (part[i][0][0][v] + part[i][0][1][v]) + (part[i][0][2][v] + part[i][0][3][v]);
            const float h1 = (part[i][1][0][v] + part[i][1][1][v]) + (part[i][1][2][v] + part[i][1][3][v]);
            if (again >> (8 * i + v) & 1) o[v] = FUSED_UP ? h / (1.0f + expf(-h)) * h1 : h;
            if (again >> (8 * i + 4 + v) & 1) o[16 + v] = h1;
        }
    }
}
// The doubtful sums of a wavefront's part of a tile: 16 rows after the other if one or two times 16 have some, else all rows, which share the
// weights' loads (d = 1024, f = 2816, 2000 rows in 16 segments: all sums doubtful, gate+up 183 -> 548, down 94 -> 304 us, 16 rows after the other 876
// and 662; an infinity in every 97th row 283 and 175; the fp32 instruction with tiles made for it 250 and 168).
template <bool FUSED_UP, bool SEG_K, int K_GROUPS>
__device__ __forceinline__ void by_f32(const GemmArgs &g, const Left<K_GROUPS> &left, int slot, int m0, int m_end, int wn, int wave, int nj, int lane) {
    const int r = lane & 15, q = lane >> 4;
    uint64_t again = 0;   // this lane's sums: bit 8 i + 4 j + v
    int need = 0;         // 16 rows of anyone's (scalar)
    for (int i = 0; i * 16 < m_end - m0; ++i) {
        const int row = i * 16 + r;
        const bool here = m0 + row < m_end && !(FUSED_UP && nj == 1 && q >= 2);
        int mine = 0;
        for (int j = 0; j < (FUSED_UP ? 1 : nj); ++j) {
            const f32x4_t sum = left.sums[wave][i * nj + j][lane];
            f32x4_t up = sum;
            if constexpr (FUSED_UP) up = nj == 2 ? left.sums[wave][i * nj + 1][lane] : left.sums[wave][i][lane ^ 32];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                bool one = doubtful(sum[v], left.a(row), left.b(wave, j * 16 + 4 * q + v), g.K);
                if constexpr (FUSED_UP) one |= doubtful(up[v], left.a(row), left.b(wave, (nj * 8 + 4 * q + v) & (B_WAVE_ROWS - 1)), g.K);
                mine |= (int)(one && here && wn + j * 16 + 4 * q + v < g.N) << (j * 4 + v);
            }
        }
        again |= (uint64_t)mine << (8 * i);
        need |= __any(mine) ? 1 << i : 0;
    }
    const FromMemory<FUSED_UP> from(g, slot, m0, wn, nj, r);
    if (__popc(need) > 2) {
        rows_by_f32<FUSED_UP, SEG_K, MAX_MF>(g, from, m0, m_end, 0, wn, lane, again);
    } else {
        for (; need; need &= need - 1) {
            const int i = __ffs(need) - 1;
            rows_by_f32<FUSED_UP, SEG_K, 1>(g, from, m0, m_end, i * 16, wn, lane, again >> (8 * i));
        }
    }
}

// MF: activation fragments of 16 rows.  NJ: weight fragments per wavefront, 2, or 1 for half a tile's weight rows (gate+up: then 8
// rows of each matrix, and the lanes of the upper half hold the up projection's sums).  SEG_K: the weights' K axis is cut in segments.
// Returns (to all lanes) whether by_f32 is to look at the wavefront's sums, which are in LDS then.
template <bool FUSED_UP, bool SEG_K, int K_GROUPS, int MF, int NJ>
__device__ __forceinline__ bool tile_body(const GemmArgs &g, int slot, int m0, int m_end, int n0, int rotation, KSegDiv seg_of, char *smem) {
    constexpr int AHEAD = MF > 3 ? 2 : 4;   // steps in flight (even)
    constexpr int AL = MF / 2;              // activation loads of 16 bytes per thread and step: 32 rows each
    constexpr bool HALF = MF % 2 != 0;      // and one of 8 bytes for the last 16 rows
    int tid = (int)threadIdx.x;
    asm volatile("" : "+v"(tid));           // what follows from it stays out of the kernel's loop over tiles
    const int group = K_GROUPS == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 8);
    tid &= 255;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, q = lane >> 4;
    const int nk = ((g.K + BK - 1) / BK + K_GROUPS - 1) / K_GROUPS;   // steps of each group
    const int k_begin = group * nk * BK, k_end = k_begin + nk * BK;
    char *const all = smem;
    smem += group * GROUP_BYTES;

    // ---- load sources (offsets without data give zeros: past the rows, past N, past K) ----
    const auto a_rsrc = rsrc_of((const char *)g.A + (int64_t)m0 * g.lda * 4);
    const int row_of = tid >> 3, chunk = tid & 7;
    uint32_t a_off[AL + 1];                  // (AL is 0 for 16 rows)
#pragma unroll
    for (int i = 0; i < AL; ++i) {
        const int row = i * 32 + row_of;
        a_off[i] = m0 + row < m_end ? (uint32_t)row * (uint32_t)(g.lda * 4) + (uint32_t)chunk * 16u : NO_DATA;
    }
    const int h_row = AL * 32 + (tid >> 4), h_chunk = tid & 15;
    const uint32_t h_off = m0 + h_row < m_end ? (uint32_t)h_row * (uint32_t)(g.lda * 4) + (uint32_t)h_chunk * 8u : NO_DATA;
    const int wn = n0 + wave * (FUSED_UP ? 8 : 16) * NJ;   // first output column of the wavefront
    const int64_t b_first = ((int64_t)slot * g.b_slot_stride + (int64_t)wn * g.ldb) * 4;
    const auto b0_rsrc = rsrc_of((const char *)g.B0 + b_first);
    const auto b1_rsrc = rsrc_of((FUSED_UP ? (const char *)g.B1 : (const char *)g.B0) + b_first);
    const int b_row = lane >> 3;
    uint32_t b_off[2 * NJ];   // FUSED_UP: the first half of the rows gate, the second up
#pragma unroll
    for (int i = 0; i < 2 * NJ; ++i) {
        const int n = FUSED_UP ? (i % NJ) * 8 + b_row : i * 8 + b_row;
        b_off[i] = wn + n < g.N ? (uint32_t)n * (uint32_t)(g.ldb * 4) + (uint32_t)chunk * 16u : NO_DATA;
    }
    char *const sb = smem + 3 * A_PLANE + wave * 3 * B_PLANE;
    // places in a plane: this thread's loads', the fragments' (16 rows, 8 lines, keep the order of the chunks)
    const int a_at = chunk_at(row_of, chunk >> 1) + (chunk & 1) * 8, h_at = chunk_at(h_row, h_chunk >> 2) + (h_chunk & 3) * 4;
    const int b_at[2] = {chunk_at(b_row, chunk >> 1) + (chunk & 1) * 8, chunk_at(8 + b_row, chunk >> 1) + (chunk & 1) * 8};
    const int frag_at = chunk_at(r, q);

    u32x2_t rh[AHEAD];
    u32x4_t ra[AHEAD][AL + 1], rb[AHEAD][2 * NJ];
    f32x4_t acc[MF][NJ], low[MF][NJ];   // sums of the products of the leading parts; of the others, 2^-8 of them and less
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = low[i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    float a_max[AL + 1], h_max = 0.0f, b_max[2 * NJ];     // largest magnitudes that this thread has seen of its rows
#pragma unroll
    for (int i = 0; i < AL; ++i) a_max[i] = 0.0f;
#pragma unroll
    for (int i = 0; i < 2 * NJ; ++i) b_max[i] = 0.0f;

    // loads of one step: K, whether there is data, then one load per slot (A: 0 .. AL - 1, the half one, B)
    int k0 = k_begin + (SEG_K ? 0 : rotation % nk * BK), left = nk, k_load = 0;   // K of the next loads and how many there are (scalar)
    uint32_t a_none = 0, h_none = 0, b_add = 0;
    auto next_loads = [&]() {
        const int k = k0 + chunk * 4;
        a_none = left > 0 && k < g.K ? 0u : NO_DATA;
        if (HALF) h_none = left > 0 && k0 + h_chunk * 2 < g.K ? 0u : NO_DATA;   // (K is a multiple of 4)
        if constexpr (SEG_K) b_add = k < g.K ? seg_of(k) * (uint32_t)((g.kseg_stride - g.kseg_len) * 4) : NO_DATA;   // (wraps past K alone)
        else b_add = a_none;
        k_load = k0 * 4;
        --left;
        k0 = SEG_K || k0 + BK != k_end ? k0 + BK : k_begin;
    };
    auto load_a = [&](int set, int i) { ra[set][i] = load16(a_rsrc, a_off[i] | a_none, (uint32_t)k_load); };
    auto load_h = [&](int set) { rh[set] = __builtin_amdgcn_raw_buffer_load_b64(a_rsrc, (int)(h_off | h_none), k_load, 0); };
    auto load_b = [&](int set, int i) {
        rb[set][i] = load16(FUSED_UP && i >= NJ ? b1_rsrc : b0_rsrc, SEG_K ? offset_with(b_off[i], b_add) : b_off[i] | b_add, (uint32_t)k_load);
    };
    // The values of a step, two at a time, in four stages of about three vector instructions; behind every second pair (or the half
    // load's one) the parts go to LDS.
    constexpr int PAIRS = 2 * AL + HALF + 4 * NJ, STAGES = 4 * PAIRS;
    float x, y;
    uint2 hi, mid, lo;
    auto stage = [&](auto number, int set, int buf) {
        constexpr int s = decltype(number)::value, pair = s / 4;
        constexpr bool is_b = pair >= 2 * AL + HALF, half = HALF && pair == 2 * AL;
        constexpr int v = is_b ? pair - 2 * AL - HALF : pair, i = half ? 0 : v >> 1;
        constexpr bool second = !half && (v & 1);
        uint32_t &h = second ? hi.y : hi.x, &m = second ? mid.y : mid.x, &l = second ? lo.y : lo.x;
        if constexpr (s % 4 == 0) {
            if constexpr (half) {
                x = __uint_as_float(rh[set][0]), y = __uint_as_float(rh[set][1]);
            } else {
                const u32x4_t w = [&]() { if constexpr (is_b) return rb[set][i]; else return ra[set][i]; }();
                x = __uint_as_float(w[second ? 2 : 0]), y = __uint_as_float(w[second ? 3 : 1]);
            }
            float &most = [&]() -> float & { if constexpr (half) return h_max; else if constexpr (is_b) return b_max[i]; else return a_max[i]; }();
            asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(most) : "v"(x), "v"(y));
            h = pack_bf16x2(x, y);
        } else if constexpr (s % 4 == 1) {
            x -= bf16_lo_to_f32(h);
            y -= bf16_hi_to_f32(h);
            // the registers are free: on to the step AHEAD of this one
            if constexpr (half) load_h(set);
            else if constexpr (second && is_b) load_b(set, i);
            else if constexpr (second) load_a(set, i);
        } else if constexpr (s % 4 == 2) {
            m = pack_bf16x2(x, y);
            x -= bf16_lo_to_f32(m);
        } else {
            y -= bf16_hi_to_f32(m);
            l = pack_bf16x2(x, y);
            char *const base = is_b ? sb + buf * BUFFER_BYTES : smem + buf * BUFFER_BYTES;
            constexpr int plane = is_b ? B_PLANE : A_PLANE;
            if constexpr (half) {
                char *const at = base + h_at;
                *(uint32_t *)at = hi.x;
                *(uint32_t *)(at + plane) = mid.x;
                *(uint32_t *)(at + 2 * plane) = lo.x;
            } else if constexpr (second) {
                char *const at = base + (is_b ? b_at[i & 1] + (i >> 1) * 16 * BK * 2 : a_at + i * 32 * BK * 2);
                *(uint2 *)at = hi;
                *(uint2 *)(at + plane) = mid;
                *(uint2 *)(at + 2 * plane) = lo;
            }
        }
    };
    // One step: LDS buffer `buf` is multiplied while the other one gets the parts of register set `set`.  A matrix instruction
    // holds its unit for 16 cycles, as long as four vector instructions theirs, and a wavefront issues in order, so the two are
    // dealt out one to one; the compiler's own order multiplies first and splits then (114 instead of 100 us, see above).
    auto step_body = [&](int buf, int set) {
        constexpr int MFMAS = PRODUCTS * MF * NJ;
        const char *const a = smem + buf * BUFFER_BYTES, *const b = sb + buf * BUFFER_BYTES;
        bf16x8_t fb[NJ][3], fa[2][2][3];
        auto read_a = [&](int f, int p) { fa[(f >> 1) & 1][f & 1][p] = *(const bf16x8_t *)(a + p * A_PLANE + f * 16 * BK * 2 + frag_at); };
#pragma unroll
        for (int p = 2; p >= 0; --p) {
#pragma unroll
            for (int j = 0; j < NJ; ++j) fb[j][p] = *(const bf16x8_t *)(b + p * B_PLANE + j * 16 * BK * 2 + frag_at);
#pragma unroll
            for (int f = 0; f < min(MF, 2); ++f) read_a(f, 2 - p);
        }
        __builtin_amdgcn_sched_barrier(0);
        // products by rounds of two activation fragments (the last one's may be one), then the smallest first
        each<MFMAS>([&](auto number) {
            constexpr int m = decltype(number)::value, f0 = m / (2 * NJ * PRODUCTS) * 2, fn = MF - f0 < 2 ? 1 : 2;
            constexpr int next = m - f0 * NJ * PRODUCTS, t = next / (fn * NJ), u = next / NJ % fn, j = next % NJ;
            f32x4_t &sum = t == PRODUCTS - 1 ? acc[f0 + u][j] : low[f0 + u][j];
            sum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j][PART_B[t]], fa[(f0 >> 1) & 1][u][PART_A[t]], sum, 0, 0, 0);
            // the next round's fragments, one read for each of the first products
            if constexpr (next < 6 && f0 + 2 + (next & 1) < MF) read_a(f0 + 2 + (next & 1), next >> 1);
            constexpr int from = (m * STAGES + MFMAS - 1) / MFMAS, to = ((m + 1) * STAGES + MFMAS - 1) / MFMAS;
            each<to - from>([&](auto n) { stage(std::integral_constant<int, from + decltype(n)::value>{}, set, buf ^ 1); });
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    // step s multiplies LDS buffer s % 2, splits and stores step s + 1's data and loads step s + 1 + AHEAD's in their place
    auto step = [&](int p) {
        next_loads();
        __builtin_amdgcn_sched_barrier(0);
        step_body(p & 1, (p + 1) % AHEAD);
        __syncthreads();
    };
#pragma unroll
    for (int p = 0; p < AHEAD; ++p) {
        next_loads();
#pragma unroll
        for (int i = 0; i < AL; ++i) load_a(p, i);
        if (HALF) load_h(p);
#pragma unroll
        for (int i = 0; i < 2 * NJ; ++i) load_b(p, i);
    }
    next_loads();
    each<STAGES>([&](auto number) { stage(number, 0, 0); });
    __syncthreads();
    int s0 = 0;
    for (; s0 + AHEAD <= nk; s0 += AHEAD) {
#pragma unroll
        for (int p = 0; p < AHEAD; ++p) step(p);
    }
#pragma unroll
    for (int p = 0; p < AHEAD - 1; ++p) {
        if (s0 + p >= nk) break;
        step(p);
    }
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] += low[i][j];

    // ---- largest magnitudes of the rows (the lanes of a row are neighbours) and the other group's sums, through LDS (the last step
    // ended with a barrier) ----
    Left<K_GROUPS> &left_here = *(Left<K_GROUPS> *)all;
    auto of_row = [&](float most, int lanes) {
#pragma unroll
        for (int o = 1; o < lanes; o <<= 1) most = fmaxf(most, __shfl_xor(most, o, 64));
        return most;
    };
#pragma unroll
    for (int i = 0; i < AL; ++i) {
        const float most = of_row(a_max[i], 8);
        if (chunk == 0) left_here.a_most[group][i * 32 + row_of] = most;
    }
    if (HALF) {
        const float most = of_row(h_max, 16);
        if (h_chunk == 0) left_here.a_most[group][h_row] = most;
    }
#pragma unroll
    for (int i = 0; i < 2 * NJ; ++i) {
        const float most = of_row(b_max[i], 8);
        if (chunk == 0) left_here.b_most[group][wave][i * 8 + b_row] = most;
    }
    [[maybe_unused]] f32x4_t *const sums = (f32x4_t *)(all + GROUP_BYTES) + (wave * MF * NJ) * 64 + lane;
    if (group != 0) {
#pragma unroll
        for (int i = 0; i < MF; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) sums[(i * NJ + j) * 64] = acc[i][j];
    }
    __syncthreads();
    if (group != 0) return false;
    float a_here[MF], b_here[NJ];   // of this lane's row and four columns of each fragment: read here, looked at when the sums are on their way out
#pragma unroll
    for (int i = 0; i < MF; ++i) a_here[i] = left_here.a(i * 16 + r);
#pragma unroll
    for (int j = 0; j < NJ; ++j) b_here[j] = left_here.b4(wave, j * 16 + 4 * q);
    if constexpr (K_GROUPS > 1) {
#pragma unroll
        for (int i = 0; i < MF; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) acc[i][j] += sums[(i * NJ + j) * 64];
    }
    // ---- epilogue: element v of lane l of a fragment is output column 4 * (l / 16) + v, row l % 16 ----
    float *const out = (float *)g.out;
#pragma unroll
    for (int i = 0; i < MF; ++i) {
        const int row = m0 + i * 16 + r;
        float up[4];
        if constexpr (FUSED_UP) {
#pragma unroll
            for (int v = 0; v < 4; ++v) up[v] = NJ == 2 ? acc[i][NJ - 1][v] : __shfl_xor(acc[i][0][v], 32, 64);
        }
        if (row >= m_end) continue;
#pragma unroll
        for (int j = 0; j < (FUSED_UP ? 1 : NJ); ++j) {
            const int col = wn + j * 16 + 4 * q;
            if (col >= g.N || (FUSED_UP && NJ == 1 && q >= 2)) continue;
            float h[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                h[v] = acc[i][j][v];
                if (FUSED_UP) h[v] = h[v] / (1.0f + expf(-h[v])) * up[v];
            }
            float *const o = out + (int64_t)row * g.ldo + col;
            if (g.N % 4 == 0) {
                *(float4 *)o = make_float4(h[0], h[1], h[2], h[3]);
            } else {
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (col + v < g.N) o[v] = h[v];
            }
        }
    }
    // Is any of the lane's sums small for its largest rows, or not finite?  (Rows of zeros give zeros, as do those past the tile's; few instructions,
    // for they are cold at the end of a tile: one test per sum took 2 us of a layer's 50 us projection.)
    float smallest = INFINITY, all_sums = 0.0f, am = 0.0f, bm = 0.0f;
#pragma unroll
    for (int j = 0; j < NJ; ++j) bm = fmaxf(bm, b_here[j]);
#pragma unroll
    for (int i = 0; i < MF; ++i) {
        float of_rows = INFINITY;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const f32x4_t &x = acc[i][j];
            const float m = fminf(fminf(fabsf(x[0]), fabsf(x[1])), fminf(fabsf(x[2]), fabsf(x[3])));
            of_rows = fminf(of_rows, b_here[j] > 0.0f ? m : INFINITY);
            all_sums += x[0];
            all_sums += x[1];
            all_sums += x[2];
            all_sums += x[3];
        }
        smallest = fminf(smallest, a_here[i] > 0.0f ? of_rows : INFINITY);
        am = fmaxf(am, a_here[i]);
    }
    const bool out_of_range = !(smallest >= least_of(am, bm, g.K)) || !(fabsf(all_sums) < INFINITY);
    if (!__any(out_of_range)) return false;
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) left_here.sums[wave][i * NJ + j][lane] = acc[i][j];
    return true;
}

// Where workgroup number b works: tile t (-1: none) of `blocks` numbers, in segment s.  SEG_PER_LANE: 1 for up to 64 row segments, 4 for
// up to 256.  Pieces of a segment have one size, and tiles are numbered and dealt to the XCDs as gemm_bf16_mid_kernel's.  Half
// tiles, and lower pieces, while there is a place for each (the places: two workgroups per compute unit, one if its groups share K).
// few_rows: most segments have no more than 16.  Gate+up projections then take tiles of 16 rows where that is enough (300 to 1200 rows in
// 64 segments, time over that of the fp32 instruction 0.985 -> 0.956, median of 752); elsewhere the code of one more height, cold in each
// launch, costs more than it saves (500 tokens, d = 548, f = 2816, layer step 144 -> 148 us), and down projections are even.
struct Place {
    int blocks, t;
    bool halves, few_rows;
    Segment s;
};
template <int SEG_PER_LANE>
__device__ __forceinline__ Place place_of(const GemmArgs &g, int b, int n_strips, int places, int lane) {
    SegTable<SEG_PER_LANE> segs;
    segs.load(g, lane);
    segs.cut(lane, BM);
    Place p;
    int more = 0, any = 0;   // segments of more than 16 rows, of any
#pragma unroll
    for (int q = 0; q < SEG_PER_LANE; ++q) {
        more += (int)__popcll(__ballot(segs.hi[q] - segs.lo[q] > 16));
        any += (int)__popcll(__ballot(segs.hi[q] > segs.lo[q]));
    }
    p.few_rows = 2 * more <= any;
    p.halves = 2 * segs.total * n_strips <= places;
    if (p.halves) {
        if (2 * segs.count(32) * n_strips <= places) segs.cut(lane, 32);
        else if (2 * segs.count(48) * n_strips <= places) segs.cut(lane, 48);
    }
    const int strips = p.halves ? 2 * n_strips : n_strips, total = segs.total * strips;
    p.blocks = (total + 63) & ~63;
    p.t = b < p.blocks ? mid::of_runs(b, total) : -1;
    p.s = Segment{0, 0, 0, 0, 1};
    if (p.t >= 0) p.s = segs.segment(p.t / strips, lane);   // (surplus workgroups leave without)
    return p;
}

template <bool FUSED_UP, bool SEG_K, int K_GROUPS>
__global__ __launch_bounds__(256 * K_GROUPS, 2 / K_GROUPS) void gemm_f32_split_kernel(const GemmArgs g, int n_strips, int n_cu) {
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    StaleRows stale;
    if (!FUSED_UP) stale = stale_rows(g);   // in flight during the work, used at the end
    const KSegDiv seg_of(SEG_K ? g.kseg_len : 2);
    for (int b = (int)blockIdx.x;;) {       // once, unless the rank has far more rows than its share
        int lane = (int)threadIdx.x & 63;
        asm volatile("" : "+v"(lane));      // the table is read again each time: kept, it would cost the tile its registers
        const int places = 2 / K_GROUPS * n_cu;
        const Place p = SEG_K || g.S <= 64 ? place_of<1>(g, b, n_strips, places, lane) : place_of<4>(g, b, n_strips, places, lane);
        if (b >= p.blocks) break;
        const bool again = b >= (int)gridDim.x;
        b += (int)gridDim.x;
        const bool more = b < p.blocks;
        if (p.t < 0) {
            if (more) continue;
            break;
        }
        const bool halves = p.halves;
        const Segment s = p.s;
        const int in_seg = p.t - s.first_tile * (halves ? 2 * n_strips : n_strips), strip = in_seg / s.tiles, piece = in_seg - strip * s.tiles;
        const int rows = ((s.hi - s.lo + s.tiles - 1) / s.tiles + 15) & ~15;
        const int m0 = s.lo + piece * rows, m_end = min(s.hi, m0 + rows);
        const int n0 = strip * (halves ? Shape<FUSED_UP>::BN / 2 : Shape<FUSED_UP>::BN);
        const int rotation = (s.slot * n_strips + (halves ? strip >> 1 : strip)) / 4;   // (of the weights alone: see above)
        if (again) __syncthreads();   // the tile before has been read
        auto tile = [&](auto nj) {
            constexpr int NJ = decltype(nj)::value;
            switch ((m_end - m0 + 15) >> 4) {
                case 1:
                    if constexpr (FUSED_UP)
                        if (p.few_rows) return tile_body<FUSED_UP, SEG_K, K_GROUPS, 1, NJ>(g, s.slot, m0, m_end, n0, rotation, seg_of, smem);
                    [[fallthrough]];
                case 2: return tile_body<FUSED_UP, SEG_K, K_GROUPS, 2, NJ>(g, s.slot, m0, m_end, n0, rotation, seg_of, smem);
                case 3: return tile_body<FUSED_UP, SEG_K, K_GROUPS, 3, NJ>(g, s.slot, m0, m_end, n0, rotation, seg_of, smem);
                case 4: return tile_body<FUSED_UP, SEG_K, K_GROUPS, 4, NJ>(g, s.slot, m0, m_end, n0, rotation, seg_of, smem);
                case 5: return tile_body<FUSED_UP, SEG_K, K_GROUPS, 5, NJ>(g, s.slot, m0, m_end, n0, rotation, seg_of, smem);
                default: return false;   // no rows
            }
        };
        if (n0 < g.N) {
            const bool look = halves ? tile(std::integral_constant<int, 1>{}) : tile(std::integral_constant<int, 2>{});
            if (look) {
                const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) & 3, nj = halves ? 1 : 2;
                by_f32<FUSED_UP, SEG_K>(g, *(const Left<K_GROUPS> *)smem, s.slot, m0, m_end, n0 + wave * (FUSED_UP ? 8 : 16) * nj, wave, nj, lane);
            }
        }
        if (!more) break;
    }
    if (FUSED_UP) share_record(g, blockIdx.x == 0); else clear_stale_rows(g, stale);
}

}  // namespace split
}  // namespace grace
