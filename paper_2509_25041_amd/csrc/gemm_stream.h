// MFMA grouped GEMM that reads both operands straight into registers: few rows per segment (decode batches, bf16 and
// fp32), and fp32 of any size whose K or tiles are too few for gemm_f32_split.h.
//
// A workgroup owns 32 weight rows of one segment (gate+up: 16 of each matrix, i.e. 16 output columns; down: 32
// columns) and up to 64 of the segment's rows, and its wavefronts split K, so that the 32 weight rows, which lie
// next to each other in memory, are read in one sweep.  A wavefront loads both operands in the layout the MFMA
// takes (row = lane % 16, 16 bytes of consecutive K at lane / 16: one v_mfma_f32_16x16x32_bf16, or four
// v_mfma_f32_16x16x4_f32 that take one of the four floats each; K is then summed in another order on both sides
// alike), DEPTH steps of 64 bytes of K ahead: no LDS, no barrier and, with buffer loads (a scalar offset that
// advances, constant lane offsets), no vector address arithmetic in the loop.  The partial sums of the
// wavefronts are added through LDS at the end, in wavefront order (deterministic).
//
// bf16, few rows: bound by HBM (the weights).  The activation rows come from L2 (every workgroup of a segment
// reads the same few), at most twice the bytes of the weights at 64 rows.  The large-tile kernel
// (gemm_bf16_persist.h) is the wrong shape there: 256 weight rows per workgroup leave most compute units without
// a tile, and a 256-row activation tile is mostly clamped duplicates.  Measured with cold weights (more than 1 GB of
// others between two uses; up / down projection, large tiles -> this kernel, us): 16 segments of d = 2048, f = 1024, 122
// rows in all of them 37.7 / 21.4 -> 29.7 / 16.4 (134 + 67 MB: 4.5 / 4.1 TB/s; a large copy moves 5.1 TB/s); a row in
// each of 4 of them 26.5 / 14.8 -> 19.3 / 10.7; 22 rows in all 16 segments of f = 768 36.1 / 19.0 -> 21.4 / 12.0.  The
// 96-row kernel takes 27.5 / 17.2, 11.7 / 8.1 and 21.7 / 13.5 there; with a third of the segments
// empty, as skewed routing leaves them, it is ahead (20.4 / 13.4 and 28.7 / 16.3), and far ahead where a few rows meet many strips (d =
// 4096, f = 14336, one segment of 64 rows 43.9 / 60.4 and 105.9 / 97.6), so gate+up projections of more than 16 tokens go there when its tiles fill the
// chip.  Register depths of 4 to 8 steps make no difference; with about 160 registers (12 wavefronts per compute unit, so
// that 1024 workgroups no longer run at once) the first case took 1.6 us more, with nt loads 3 us more.
//
// fp32, any number of rows: d = 1024, f = 2816, 8 segments and 977 rows in all, up / down projection 351 / 492 us on the
// vector ALUs -> 175 / 108 us (64 / 52 TFLOP/s; the matrix cores are busy 45 % of the time).  What bounds it is the
// address unit: in the MFMA's layout consecutive lanes lie in different rows, so a load touches a line per lane.
// Register depths of 3 and 4 steps change nothing, pieces of 32 rows take 198 / 116 us; staged through LDS 156 / 96 us, on the
// bf16 matrix cores about 105 / 80 us (gemm_f32_split.h).  Wavefronts that start at different steps of their part of K, as the 96-row kernel's tiles do, are even (16
// tokens, 12.8 / 7.8 -> 12.4 / 8.2 us).  Error against 64 bits
// 6.4e-7, half of the vector kernel's 1.3e-6 (shorter chains of additions).
#pragma once
#include <type_traits>

#include "bf16.h"
#include "gemm_common.h"

namespace grace {
namespace strm {

constexpr int MAX_ROWS = 64;      // rows a workgroup handles at a time; bf16: rows per segment up to which this kernel is used
constexpr int STEP_BYTES = 64;    // of K, per row
constexpr int MAX_WAVES = 16;     // per workgroup; also keeps the kernel at 128 registers = 16 wavefronts per compute unit

// EL: bytes per element, 2 (bf16) or 4 (fp32)
template <int EL>
constexpr int kstep() { return STEP_BYTES / EL; }

template <bool FUSED_UP>
struct Shape {
    static constexpr int COLS = FUSED_UP ? 16 : 32;   // output columns per workgroup
};

// LDS bytes of `waves` wavefronts' partial sums (2 weight fragments x mf activation fragments x 1 KB)
inline int lds_bytes(int waves, int mf) { return waves * mf * 2 * 1024; }

// The rows that a workgroup handles at a time: output rows [m0, m_end), activation rows from a0 on, or those that `list` (LDS) names.
struct RowsOf {
    int m0, m_end, a0;
    const int16_t *list;
};

// MF: activation fragments of 16 rows the workgroup handles at a time
template <bool FUSED_UP, int EL, int MF, bool LISTED>
__device__ __forceinline__ void rows_body(const GemmArgs &g, int slot, const RowsOf &rows, int n0, float4 *red) {
    const int m0 = rows.m0, m_end = rows.m_end;
    constexpr int KSTEP = kstep<EL>();
    constexpr int DEPTH = MF == 1 ? 6 : MF == 2 ? 4 : MF == 3 ? 3 : 2;   // what 128 registers hold
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), waves = (int)blockDim.x >> 6;
    const int r = lane & 15, q = lane >> 4;
    const int n_steps = g.K / KSTEP;                          // whole steps; the rest below
    const int s0 = wave * n_steps / waves, n = (wave + 1) * n_steps / waves - s0;

    // lane offsets (bytes) of the fragments
    uint32_t a_off[MF], b_off[2];
#pragma unroll
    for (int i = 0; i < MF; ++i) {
        const int m = min(i * 16 + r, m_end - m0 - 1);
        a_off[i] = (uint32_t)(LISTED ? rows.list[m] : m) * (uint32_t)(g.lda * EL) + (uint32_t)q * 16u;
    }
    {
        const int na = min(n0 + r, g.N - 1), nb = FUSED_UP ? na : min(n0 + 16 + r, g.N - 1);
        b_off[0] = (uint32_t)(na - n0) * (uint32_t)(g.ldb * EL) + (uint32_t)q * 16u;
        b_off[1] = (uint32_t)(nb - n0) * (uint32_t)(g.ldb * EL) + (uint32_t)q * 16u;
    }
    const int64_t b_first = ((int64_t)slot * g.b_slot_stride + (int64_t)n0 * g.ldb) * EL;
    const auto a_rsrc = rsrc_of((const char *)g.A + (LISTED ? 0 : (int64_t)rows.a0 * g.lda * EL));
    const auto b0_rsrc = rsrc_of((const char *)g.B0 + b_first);
    const auto b1_rsrc = rsrc_of((FUSED_UP ? (const char *)g.B1 : (const char *)g.B0) + b_first);
    // scalar offsets along K; the weights' jumps at the ends of K segments (of a length that is a multiple of the
    // step where there are several)
    int kpos = s0 * KSTEP;
    uint32_t a_k = (uint32_t)(kpos * EL), b_k = (uint32_t)((kpos < g.kseg_len ? kpos : koff(g, kpos)) * EL);
    kpos = kpos < g.kseg_len ? kpos : kpos % g.kseg_len;

    u32x4_t ra[DEPTH][MF], rb[DEPTH][2];
    f32x4_t acc[MF][2];
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};

    auto load = [&](int p) {
        rb[p][0] = load16(b0_rsrc, b_off[0], b_k);
        rb[p][1] = load16(b1_rsrc, b_off[1], b_k);
#pragma unroll
        for (int i = 0; i < MF; ++i) ra[p][i] = load16(a_rsrc, a_off[i], a_k);
        __builtin_amdgcn_sched_barrier(0);   // the loads stay DEPTH steps ahead of their use
        a_k += STEP_BYTES;
        b_k += STEP_BYTES;
        kpos += KSTEP;
        if (kpos == g.kseg_len) {
            kpos = 0;
            b_k += (uint32_t)((g.kseg_stride - g.kseg_len) * EL);
        }
    };
    auto mma = [&](int p) {
        if constexpr (EL == 2) {
#pragma unroll
            for (int i = 0; i < MF; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, rb[p][j]),
                                                                        __builtin_bit_cast(bf16x8_t, ra[p][i]), acc[i][j], 0, 0, 0);
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int i = 0; i < MF; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(rb[p][j][v]), __uint_as_float(ra[p][i][v]),
                                                                         acc[i][j], 0, 0, 0);
        }
    };
    // Steps 0 .. n-1 through a ring of DEPTH register sets: step i is followed by the loads of step i + DEPTH
    // into the registers it has freed.
    if (n >= DEPTH) {
#pragma unroll
        for (int p = 0; p < DEPTH; ++p) load(p);
        int i0 = 0;
        for (; i0 + 2 * DEPTH <= n; i0 += DEPTH) {
#pragma unroll
            for (int p = 0; p < DEPTH; ++p) {
                mma(p);
                load(p);
            }
        }
        const int more = n - i0 - DEPTH;   // loads still to be issued, fewer than DEPTH
#pragma unroll
        for (int p = 0; p < DEPTH - 1; ++p) {
            if (p >= more) break;
            mma(p);
            load(p);
        }
#pragma unroll
        for (int p = 0; p < DEPTH; ++p) mma(p);
    } else {
#pragma unroll
        for (int p = 0; p < DEPTH - 1; ++p)
            if (p < n) load(p);
#pragma unroll
        for (int p = 0; p < DEPTH - 1; ++p)
            if (p < n) mma(p);
    }
    if (n_steps * KSTEP < g.K && wave == waves - 1) {
        // the last wavefront takes what is left of K (a multiple of 16 bytes), zeros past the end
        const int k = n_steps * KSTEP;
        const bool in = k + q * (16 / EL) < g.K;
        const uint32_t kb = (uint32_t)(koff(g, k) * EL);
        rb[0][0] = load16(b0_rsrc, in ? b_off[0] : NO_DATA, kb);
        rb[0][1] = load16(b1_rsrc, in ? b_off[1] : NO_DATA, kb);
#pragma unroll
        for (int i = 0; i < MF; ++i) ra[0][i] = load16(a_rsrc, in ? a_off[i] : NO_DATA, (uint32_t)(k * EL));
        mma(0);
    }

    // ---- add the wavefronts' sums, activation on the result ----
    // element v of lane l of a fragment: output column 4 * (l / 16) + v, row l % 16
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
            red[((wave * MF + i) * 2 + j) * 64 + lane] = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
    __syncthreads();
    auto total = [&](int i, int j, int l) {
        float4 s = red[(i * 2 + j) * 64 + l];
        for (int w = 1; w < waves; ++w) {
            const float4 v = red[((w * MF + i) * 2 + j) * 64 + l];
            s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
        }
        return s;
    };
    for (int it = tid; it < MF * (FUSED_UP ? 64 : 128); it += (int)blockDim.x) {
        const int l = it & 63, i = FUSED_UP ? it >> 6 : it >> 7, j = FUSED_UP ? 0 : (it >> 6) & 1;
        const int row = m0 + i * 16 + (l & 15), col = n0 + j * 16 + 4 * (l >> 4);
        if (row >= m_end || col >= g.N) continue;
        float4 h = total(i, j, l);
        if (FUSED_UP) {
            const float4 u = total(i, 1, l);
            auto silu = [](float x) { return EL == 2 ? x * __frcp_rn(1.0f + __expf(-x)) : x / (1.0f + expf(-x)); };
            h.x = silu(h.x) * u.x;
            h.y = silu(h.y) * u.y;
            h.z = silu(h.z) * u.z;
            h.w = silu(h.w) * u.w;
        }
        const int64_t o = (int64_t)row * g.ldo + col;
        if constexpr (EL == 2) {   // N is a multiple of 8
            *(uint2 *)((uint16_t *)g.out + o) = make_uint2(pack_bf16x2(h.x, h.y), pack_bf16x2(h.z, h.w));
        } else if (g.N % 4 == 0) {
            *(float4 *)((float *)g.out + o) = h;
        } else {
            float *out = (float *)g.out + o;
            out[0] = h.x;
            if (col + 1 < g.N) out[1] = h.y;
            if (col + 2 < g.N) out[2] = h.z;
            if (col + 3 < g.N) out[3] = h.w;
        }
    }
}

// rows_body with as many fragments as the rows need, at most MF_MAX
template <bool FUSED_UP, int EL, int MF_MAX, bool LISTED = false>
__device__ __forceinline__ void rows_any(const GemmArgs &g, int slot, const RowsOf &of, int n0, float4 *red) {
    const int rows = of.m_end - of.m0;
    if (MF_MAX == 1 || rows <= 16) rows_body<FUSED_UP, EL, 1, LISTED>(g, slot, of, n0, red);
    else if (MF_MAX == 2 || rows <= 32) rows_body<FUSED_UP, EL, MF_MAX < 2 ? MF_MAX : 2, LISTED>(g, slot, of, n0, red);
    else if (rows <= 48) rows_body<FUSED_UP, EL, MF_MAX < 3 ? MF_MAX : 3, LISTED>(g, slot, of, n0, red);
    else rows_body<FUSED_UP, EL, MF_MAX, LISTED>(g, slot, of, n0, red);
}

// One workgroup per (segment, strip of weight rows): block = slot * n_strips + strip.  MF_MAX: fragments of 16
// rows that cover the launcher's bound on a segment's rows; a segment with fewer rows takes a shorter
// body, one with more is walked in pieces.
template <bool FUSED_UP, int EL, int MF_MAX>
__global__ __launch_bounds__(64 * MAX_WAVES) void gemm_stream_kernel(const GemmArgs g, int n_strips) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int slot = (int)blockIdx.x / n_strips, n0 = ((int)blockIdx.x - slot * n_strips) * Shape<FUSED_UP>::COLS;
    StaleRows stale;
    if (!FUSED_UP) stale = stale_rows(g);
    const int lo = __builtin_amdgcn_readfirstlane(g.seg_off ? g.seg_off[slot] : 0);
    const int hi = __builtin_amdgcn_readfirstlane(g.seg_off ? g.seg_off[slot + 1] : g.M_single);
    for (int m0 = lo; m0 < hi; m0 += MF_MAX * 16) {
        if (m0 > lo) __syncthreads();   // the sums of the rows before have been read
        rows_any<FUSED_UP, EL, MF_MAX>(g, slot, {m0, min(hi, m0 + MF_MAX * 16), activation_row(g, slot, lo, m0), nullptr}, n0, (float4 *)smem);
    }
    if (FUSED_UP) share_record(g, blockIdx.x == 0); else clear_stale_rows(g, stale);
}

// One workgroup per (segment, strip of weight rows, piece of at most MAX_ROWS of the segment's rows), pieces of
// one size (a multiple of 16) per segment.  Numbered by segment, strip, piece, and cut into eight equal ranges,
// one per XCD (workgroups are dealt to the XCDs round-robin): the workgroups that run together on an XCD share
// weight strips and rows in its L2.  The grid covers the launcher's bound on the pieces; the rest exits.
// Where all pieces leave three in four of the compute units (or every other one) without work, they have 16 (32)
// rows: a piece of 64 keeps its matrix cores busy for several times as long, on the few that have one (12 tiles, 129 rows of 2 segments, K = 256, N = 128
// 8.8 -> 6.7 us; layer steps, two or four slots, d = 128, f = 256, 65 to 700 tokens 1.03 to 1.16 times as fast, f = 1024 1.08 to 1.28, d = 512, f = 256 0.99 to
// 1.20; more slots or d = 1024, where it seldom applies, 0.99 to 1.20).
template <bool FUSED_UP, int EL, int SEG_PER_LANE>
__global__ __launch_bounds__(256, 4) void gemm_stream_tiles_kernel(const GemmArgs g, int n_strips, int n_cu) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int lane = (int)threadIdx.x & 63;
    if (FUSED_UP) share_record(g, blockIdx.x == 0); else share_clear_stale(g);
    SegTable<SEG_PER_LANE> segs;
    segs.load(g, lane);
    segs.cut(lane, MAX_ROWS);
    if (4 * segs.total * n_strips <= n_cu) segs.cut(lane, MAX_ROWS / 4);
    else if (2 * segs.total * n_strips <= n_cu) segs.cut(lane, MAX_ROWS / 2);
    const int total = segs.total * n_strips, xcd = (int)blockIdx.x & 7, j = (int)blockIdx.x >> 3;
    const int each = total >> 3, rem = total & 7;
    if (j >= each + (xcd < rem ? 1 : 0)) return;
    const int t = xcd * each + min(xcd, rem) + j;
    const Segment s = segs.segment(t / n_strips, lane);
    const int in_seg = t - s.first_tile * n_strips, strip = in_seg / s.tiles, piece = in_seg - strip * s.tiles;
    const int rows = ((s.hi - s.lo + s.tiles - 1) / s.tiles + 15) & ~15;
    const int m0 = s.lo + piece * rows;
    if (m0 < s.hi)
        rows_any<FUSED_UP, EL, MAX_ROWS / 16>(g, s.slot, {m0, min(s.hi, m0 + rows), activation_row(g, s.slot, s.lo, m0), nullptr},
                                              strip * Shape<FUSED_UP>::COLS, (float4 *)smem);
}

}  // namespace strm
}  // namespace grace
