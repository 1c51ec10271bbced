// fp32 grouped GEMM on the matrix cores (v_mfma_f32_16x16x4_f32: full fp32 products and sums) for long launches of batches of
// more than 64 tokens: 96 rows x 64 weight rows per workgroup, K a multiple of 4.  Short ones, whose few tiles leave units idle
// or waiting for the last, are faster on the streaming kernel (mid_f32_is_faster in ffn.hip).
//
// The same staging as gemm_bf16_mid.h: whole 128-byte lines into registers AHEAD steps ahead, then one of two LDS
// buffers, one barrier per step of 32 K.  A lane reads 16 bytes, four consecutive K, of a row and four MFMAs take one of them each (K
// is summed in another order on both sides alike), into four accumulators, which are added at the end: chains of K / 16
// additions as short as the streaming kernel's, whose wavefronts split K.  With loads in the MFMA's own layout (that
// kernel) the address unit is the bound, 45 % of the matrix cores' time; here a step's 32 cycles per MFMA are far longer than
// its loads, so what bounds it is the matrix cores and how evenly the tiles fall on the compute units: 64 weight rows
// per workgroup, not 128, and pieces of up to 96 rows, lower ones while they leave units without work.
// d = 1024, f = 2816, 8 segments, 977 rows, streaming kernel -> this one: gate+up 175 -> 156, down 107 -> 96 us (64 -> 72 and
// 52 -> 59 TFLOP/s; a single segment of 6144 rows 110 and 123, the library 151).  The rest is the tiles' uneven sizes on few compute
// units: 658 rows in seven full pieces, 9 to 30 rows in others.
#pragma once
#include "gemm_bf16_mid.h"

namespace grace {
namespace midf {

constexpr int BM = 96, BK = 32, THREADS = 256;
constexpr int A_BYTES = BM * mid::ROW_BYTES, B_WAVE_BYTES = 16 * mid::ROW_BYTES, LDS_BYTES = 2 * A_BYTES + 8 * B_WAVE_BYTES;
static_assert(BK * 4 == mid::ROW_BYTES, "a step is one line per row");

template <bool FUSED_UP>
struct Shape {
    static constexpr int BN = FUSED_UP ? 32 : 64;    // output columns per workgroup
};

// MF: activation fragments of 16 rows.  SEG_K: the weights' K axis is cut in segments.
template <bool FUSED_UP, bool SEG_K, int MF>
__device__ __forceinline__ void tile_body(const GemmArgs &g, int slot, int m0, int m_end, int n0, int first_step, char *smem) {
    constexpr int AHEAD = MF > 4 ? 2 : 4;   // steps in flight (even)
    constexpr int AL = (MF + 1) / 2;        // activation loads per thread and step: 32 rows each
    int tid = (int)threadIdx.x;
    asm volatile("" : "+v"(tid));           // what follows from it stays out of the kernel's loop over tiles
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, q = lane >> 4;
    const int nk = (g.K + BK - 1) / BK, k_end = nk * BK;

    // ---- load sources (offsets without data give zeros: past the rows, past N, past K) ----
    const auto a_rsrc = rsrc_of((const char *)g.A + (int64_t)m0 * g.lda * 4);
    const int row_of = tid >> 3, chunk = tid & 7;
    uint32_t a_off[AL];
#pragma unroll
    for (int i = 0; i < AL; ++i) {
        const int row = i * 32 + row_of;
        a_off[i] = m0 + row < m_end ? (uint32_t)row * (uint32_t)(g.lda * 4) + (uint32_t)chunk * 16u : NO_DATA;
    }
    const int wn = n0 + wave * (FUSED_UP ? 8 : 16);   // first output column of the wavefront
    const int64_t b_first = ((int64_t)slot * g.b_slot_stride + (int64_t)wn * g.ldb) * 4;
    const auto b0_rsrc = rsrc_of((const char *)g.B0 + b_first);
    const auto b1_rsrc = rsrc_of((FUSED_UP ? (const char *)g.B1 : (const char *)g.B0) + b_first);
    const int b_row = lane >> 3;
    uint32_t b_off[2];   // FUSED_UP: 8 rows of each matrix
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int n = FUSED_UP ? b_row : i * 8 + b_row;
        b_off[i] = wn + n < g.N ? (uint32_t)n * (uint32_t)(g.ldb * 4) + (uint32_t)chunk * 16u : NO_DATA;
    }
    char *sb = smem + 2 * A_BYTES + wave * 2 * B_WAVE_BYTES;
    KSegWalk walk{chunk * 4};

    u32x4_t ra[AHEAD][AL], rb[AHEAD][2];
    f32x4_t acc[4][MF];
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int i = 0; i < MF; ++i) acc[v][i] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};

    int k0 = first_step * BK, left = nk;   // K of the next loads and how many there are (scalar)
    auto load = [&](int set) {
        const int k = k0 + chunk * 4;
        const uint32_t none = left > 0 && k < g.K ? 0u : NO_DATA;
        const uint32_t add = SEG_K ? walk.next(k, g.K, g.kseg_len, g.kseg_stride, BK, 4) : none;
#pragma unroll
        for (int i = 0; i < AL; ++i) ra[set][i] = load16(a_rsrc, a_off[i] | none, (uint32_t)k0 * 4u);
#pragma unroll
        for (int i = 0; i < 2; ++i)
            rb[set][i] = load16(i ? b1_rsrc : b0_rsrc, SEG_K ? offset_with(b_off[i], add) : b_off[i] | add, (uint32_t)k0 * 4u);
        --left;
        k0 = SEG_K || k0 + BK != k_end ? k0 + BK : 0;
    };
    auto store = [&](int set, int buf) {
#pragma unroll
        for (int i = 0; i < AL; ++i) *(u32x4_t *)(smem + buf * A_BYTES + mid::chunk_at(i * 32 + row_of, chunk)) = ra[set][i];
#pragma unroll
        for (int i = 0; i < 2; ++i) *(u32x4_t *)(sb + buf * B_WAVE_BYTES + mid::chunk_at(i * 8 + b_row, chunk)) = rb[set][i];
    };
    // Two groups of 16 K; the second group's activation fragment i is read into the registers of the first group's when
    // that has been multiplied.
    f32x4_t fa[MF], fb[2];
    auto compute = [&](int buf) {
        auto read_a = [&](int i, int gk) { fa[i] = *(const f32x4_t *)(smem + buf * A_BYTES + mid::chunk_at(i * 16 + r, gk * 4 + q)); };
        auto mma = [&](int i, int gk) {
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[v][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[gk][v], fa[i][v], acc[v][i], 0, 0, 0);
        };
#pragma unroll
        for (int gk = 0; gk < 2; ++gk) fb[gk] = *(const f32x4_t *)(sb + buf * B_WAVE_BYTES + mid::chunk_at(r, gk * 4 + q));
#pragma unroll
        for (int i = 0; i < MF; ++i) read_a(i, 0);
#pragma unroll
        for (int i = 0; i < MF; ++i) {
            mma(i, 0);
            read_a(i, 1);
        }
#pragma unroll
        for (int i = 0; i < MF; ++i) mma(i, 1);
        __builtin_amdgcn_sched_group_barrier(0x100, MF + 2, 0);   // LDS reads
#pragma unroll
        for (int i = 0; i < MF; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);    // MFMA
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 4 * MF, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    // step s multiplies LDS buffer s % 2, stores step s + 1's data and loads step s + AHEAD's
    auto step = [&](int p) {
        load(p);
        __builtin_amdgcn_sched_barrier(0);
        compute(p & 1);
        store((p + 1) % AHEAD, (p + 1) & 1);
        __syncthreads();
    };
#pragma unroll
    for (int p = 0; p < AHEAD; ++p) load(p);
    store(0, 0);
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

    // ---- epilogue: element v of lane l of a fragment is weight row 4 * (l / 16) + v, row l % 16 ----
#pragma unroll
    for (int i = 0; i < MF; ++i) {
        const int row = m0 + i * 16 + r, col = wn + 4 * q;
        float h[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            h[v] = (acc[0][i][v] + acc[1][i][v]) + (acc[2][i][v] + acc[3][i][v]);
            if (FUSED_UP) {   // the lanes of the upper half hold the up projection's sums
                const float up = __shfl_xor(h[v], 32, 64);
                h[v] = h[v] / (1.0f + expf(-h[v])) * up;
            }
        }
        if (row < m_end && col < g.N && !(FUSED_UP && q >= 2))   // N is a multiple of 4
            *(float4 *)((float *)g.out + (int64_t)row * g.ldo + col) = make_float4(h[0], h[1], h[2], h[3]);
    }
}

// SEG_PER_LANE: 1 for up to 64 row segments, 4 for up to 256.  Grid and numbering as gemm_bf16_mid_kernel's whole tiles;
// pieces of 16, 32 or 64 rows while there is a compute unit for each.
template <bool FUSED_UP, bool SEG_K, int SEG_PER_LANE>
__global__ __launch_bounds__(THREADS, 2) void gemm_f32_mid_kernel(const GemmArgs g, int n_strips, int n_cu) {
    __shared__ __attribute__((aligned(1024))) char smem[LDS_BYTES];
    StaleRows stale;
    if (!FUSED_UP) stale = stale_rows(g);   // in flight during the work, used at the end
    for (int b = (int)blockIdx.x;;) {       // once, unless the rank has far more rows than its share
        int lane = (int)threadIdx.x & 63;
        asm volatile("" : "+v"(lane));      // the table is read again each time: kept, it would cost the tile its registers
        SegTable<SEG_PER_LANE> segs;
        segs.load(g, lane);
        segs.cut(lane, BM);
        if (segs.total * n_strips <= n_cu) {
            if (segs.count(16) * n_strips <= n_cu) segs.cut(lane, 16);
            else if (segs.count(32) * n_strips <= n_cu) segs.cut(lane, 32);
            else if (segs.count(64) * n_strips <= n_cu) segs.cut(lane, 64);
        }
        const int total = segs.total * n_strips;
        const int blocks = (total + 63) & ~63;
        if (b >= blocks) break;
        const int t = mid::of_runs(b, total);
        const bool again = b >= (int)gridDim.x;
        b += (int)gridDim.x;
        const bool more = b < blocks;
        if (t < 0) {
            if (more) continue;
            break;
        }
        const Segment s = segs.segment(t / n_strips, lane);
        const int in_seg = t - s.first_tile * n_strips, strip = in_seg / s.tiles, piece = in_seg - strip * s.tiles;
        const int rows = ((s.hi - s.lo + s.tiles - 1) / s.tiles + 15) & ~15;
        const int m0 = s.lo + piece * rows, m_end = min(s.hi, m0 + rows), n0 = strip * Shape<FUSED_UP>::BN;
        const int first_step = SEG_K ? 0 : (s.slot * n_strips + strip) / 4 % ((g.K + BK - 1) / BK);
        if (again) __syncthreads();   // the tile before has been read
        switch ((m_end - m0 + 15) >> 4) {
            case 1: tile_body<FUSED_UP, SEG_K, 1>(g, s.slot, m0, m_end, n0, first_step, smem); break;
            case 2: tile_body<FUSED_UP, SEG_K, 2>(g, s.slot, m0, m_end, n0, first_step, smem); break;
            case 3: tile_body<FUSED_UP, SEG_K, 3>(g, s.slot, m0, m_end, n0, first_step, smem); break;
            case 4: tile_body<FUSED_UP, SEG_K, 4>(g, s.slot, m0, m_end, n0, first_step, smem); break;
            case 5: tile_body<FUSED_UP, SEG_K, 5>(g, s.slot, m0, m_end, n0, first_step, smem); break;
            case 6: tile_body<FUSED_UP, SEG_K, 6>(g, s.slot, m0, m_end, n0, first_step, smem); break;
            default: break;   // no rows
        }
        if (!more) break;
    }
    if (FUSED_UP) share_record(g); else clear_stale_rows(g, stale);
}

}  // namespace midf
}  // namespace grace
