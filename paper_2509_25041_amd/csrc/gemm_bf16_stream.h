// bf16 MFMA grouped GEMM for a few rows per segment (decode batches): streams the weights.
//
// With at most MAX_ROWS rows per segment the product is bound by reading every weight once.  The
// large-tile kernel (gemm_bf16_persist.h) is then the wrong shape: 256 weight rows per workgroup leave
// most compute units without a tile, a 256-row activation tile is mostly clamped duplicates, and
// one workgroup per compute unit has too few bytes in flight.  Here a workgroup owns 32 weight rows of
// one segment (gate+up: 16 of each matrix, i.e. 16 output columns; down: 32 columns) and its wavefronts
// split K, so that the 32 rows, which lie next to each other in memory, are read in one sweep.  A
// wavefront loads both operands straight into registers in the layout v_mfma_f32_16x16x32_bf16 takes
// (row = lane % 16, 8 consecutive K = 16 bytes at lane / 16), DEPTH steps of 32 K ahead: no LDS, no
// barrier and no address arithmetic in the loop.  The partial sums of the wavefronts are added through
// LDS at the end, in wavefront order (deterministic).
//
// The activation rows come from L2 (every workgroup of a segment reads the same few), at most twice the
// bytes of the weights at 64 rows.
//
// Bound: HBM (the weights).  Measured (up / down projection, large-tile kernel before -> this one): 16 segments
// of d = 2048, f = 1024 and 122 rows in all 38.1 / 22.0 -> 28.8 / 16.8 us (134 + 67 MB: 4.7 / 4.0 TB/s; a large
// copy moves 5.1 TB/s); 4 rows in 4 segments 26.4 / 15.3 -> 8.2 / 5.1 us; 22 rows in 16 segments of f = 768
// 27.4 / 13.3 -> 12.0 / 8.2 us.  Register depths of 4 to 8 steps make no difference; with about 160 registers (12
// wavefronts per compute unit, so that 1024 workgroups no longer run at once) the first case took 30.4 us, with
// nt loads 3 us more.
#pragma once
#include "bf16.h"
#include "gemm_common.h"

namespace grace {
namespace strm {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;

constexpr int MAX_ROWS = 64;      // rows per segment up to which this kernel is used
constexpr int KSTEP = 32;
constexpr int MAX_WAVES = 16;     // per workgroup; also keeps the kernel at 128 registers = 16 wavefronts per compute unit

template <bool FUSED_UP>
struct Shape {
    static constexpr int COLS = FUSED_UP ? 16 : 32;   // output columns per workgroup
};

// LDS bytes of `waves` wavefronts' partial sums (2 weight fragments x mf activation fragments x 1 KB)
inline int lds_bytes(int waves, int mf) { return waves * mf * 2 * 1024; }

// The loads of one K step, issued without waiting: two weight fragments and MF activation fragments of 16
// bytes per lane, each from a scalar base and a lane offset.  To the compiler the registers hold their
// values at once; wait_loads below is what makes that true before they are used.  s_nop 4: the wait states
// between a vector instruction that wrote one of the scalar registers and the load that reads it, which
// the compiler cannot keep for an assembly block.
template <int MF>
__device__ __forceinline__ void issue_loads(u32x4_t (&a)[MF], u32x4_t (&b)[2], const char *pa, const char *pb0, const char *pb1,
                                            const uint32_t (&a_off)[MF], const uint32_t (&b_off)[2]) {
    asm volatile("s_nop 4\n\tglobal_load_dwordx4 %0, %2, %4\n\tglobal_load_dwordx4 %1, %3, %5"
                 : "+v"(b[0]), "+v"(b[1]) : "v"(b_off[0]), "v"(b_off[1]), "s"(pb0), "s"(pb1) : "memory");
#pragma unroll
    for (int i = 0; i < MF; ++i) asm volatile("s_nop 4\n\tglobal_load_dwordx4 %0, %1, %2" : "+v"(a[i]) : "v"(a_off[i]), "s"(pa) : "memory");
}
// all but the newest NEWER loads of this wavefront have landed; the step's registers pass through, so that
// their uses stay behind the wait
template <int NEWER, int MF>
__device__ __forceinline__ void wait_loads(u32x4_t (&a)[MF], u32x4_t (&b)[2]) {
    asm volatile("s_waitcnt vmcnt(%2)" : "+v"(b[0]), "+v"(b[1]) : "n"(NEWER) : "memory");
#pragma unroll
    for (int i = 0; i < MF; ++i) asm volatile("" : "+v"(a[i]));
}

// MF: activation fragments of 16 rows the workgroup handles at a time
template <bool FUSED_UP, int MF>
__device__ __forceinline__ void rows_body(const GemmArgs &g, int slot, int m0, int m_end, int n0, float4 *red) {
        constexpr int DEPTH = MF == 1 ? 6 : MF == 2 ? 4 : MF == 3 ? 3 : 2;   // what 128 registers hold
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), waves = (int)blockDim.x >> 6;
    const int r = lane & 15, q = lane >> 4;
    const int n_steps = g.K / KSTEP;                          // whole steps; the rest below
    const int s0 = wave * n_steps / waves, n = (wave + 1) * n_steps / waves - s0;

    // lane offsets (bytes) of the fragments from scalar bases that advance along K
    uint32_t a_off[MF], b_off[2];
#pragma unroll
    for (int i = 0; i < MF; ++i) {
        const int m = min(m0 + i * 16 + r, m_end - 1);
        a_off[i] = (uint32_t)(m - m0) * (uint32_t)(g.lda * 2) + (uint32_t)q * 16u;
    }
    {
        const int na = min(n0 + r, g.N - 1), nb = FUSED_UP ? na : min(n0 + 16 + r, g.N - 1);
        b_off[0] = (uint32_t)(na - n0) * (uint32_t)(g.ldb * 2) + (uint32_t)q * 16u;
        b_off[1] = (uint32_t)(nb - n0) * (uint32_t)(g.ldb * 2) + (uint32_t)q * 16u;
    }
    const char *a_base = (const char *)g.A + (int64_t)m0 * g.lda * 2;
    const int64_t b_first = ((int64_t)slot * g.b_slot_stride + (int64_t)n0 * g.ldb) * 2;
    const char *b_base0 = (const char *)g.B0 + b_first, *b_base1 = (FUSED_UP ? (const char *)g.B1 : (const char *)g.B0) + b_first;
    // weight K position: segments of kseg_len (a multiple of the step where there are several)
    int kpos = s0 * KSTEP;
    const char *pa = a_base + (int64_t)kpos * 2;
    const int64_t bo = kpos < g.kseg_len ? kpos : koff(g, kpos);
    const char *pb0 = b_base0 + bo * 2, *pb1 = b_base1 + bo * 2;
    kpos = kpos < g.kseg_len ? kpos : kpos % g.kseg_len;

    u32x4_t ra[DEPTH][MF], rb[DEPTH][2];
    f32x4_t acc[MF][2];
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int p = 0; p < DEPTH; ++p) {
        rb[p][0] = rb[p][1] = u32x4_t{0u, 0u, 0u, 0u};
#pragma unroll
        for (int i = 0; i < MF; ++i) ra[p][i] = u32x4_t{0u, 0u, 0u, 0u};
    }

    auto load = [&](int p) {
        issue_loads<MF>(ra[p], rb[p], pa, pb0, pb1, a_off, b_off);
        int64_t step = KSTEP * 2;
        pa += step;
        kpos += KSTEP;
        if (kpos == g.kseg_len) {
            kpos = 0;
            step += (g.kseg_stride - g.kseg_len) * 2;
        }
        pb0 += step;
        pb1 += step;
    };
    auto mma = [&](int p) {
#pragma unroll
        for (int i = 0; i < MF; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, rb[p][j]),
                                                                    __builtin_bit_cast(bf16x8_t, ra[p][i]), acc[i][j], 0, 0, 0);
    };
    // Steps 0 .. n-1 through a ring of DEPTH register sets.  Step i waits for its own loads only and is
    // followed by the loads of step i + DEPTH into the registers it has freed; once there are none left to
    // issue, one wait covers all that remains.
    constexpr int NEWER = (DEPTH - 1) * (2 + MF);
    if (n >= DEPTH) {
#pragma unroll
        for (int p = 0; p < DEPTH; ++p) load(p);
        int i0 = 0;
        for (; i0 + 2 * DEPTH <= n; i0 += DEPTH) {
#pragma unroll
            for (int p = 0; p < DEPTH; ++p) {
                wait_loads<NEWER, MF>(ra[p], rb[p]);
                mma(p);
                load(p);
            }
        }
        const int more = n - i0 - DEPTH;   // loads still to be issued, fewer than DEPTH
#pragma unroll
        for (int p = 0; p < DEPTH - 1; ++p) {
            if (p >= more) break;
            wait_loads<NEWER, MF>(ra[p], rb[p]);
            mma(p);
            load(p);
        }
#pragma unroll
        for (int p = 0; p < DEPTH; ++p) {
            wait_loads<0, MF>(ra[p], rb[p]);
            mma(p);
        }
    } else {
#pragma unroll
        for (int p = 0; p < DEPTH - 1; ++p)
            if (p < n) load(p);
#pragma unroll
        for (int p = 0; p < DEPTH - 1; ++p) {
            wait_loads<0, MF>(ra[p], rb[p]);
            if (p < n) mma(p);
        }
    }
    if (n_steps * KSTEP < g.K && wave == waves - 1) {
        // K is a multiple of 8: the last wavefront takes what is left of it, zeros past the end
        const int k = n_steps * KSTEP + q * 8;
        const bool in = k < g.K;
        const int64_t kb = in ? koff(g, k) : 0;
        const uint32_t qo = (uint32_t)q * 16u;
        const u32x4_t zero = {0u, 0u, 0u, 0u};
        rb[0][0] = in ? *(const u32x4_t *)(b_base0 + (b_off[0] - qo) + kb * 2) : zero;
        rb[0][1] = in ? *(const u32x4_t *)(b_base1 + (b_off[1] - qo) + kb * 2) : zero;
#pragma unroll
        for (int i = 0; i < MF; ++i) ra[0][i] = in ? *(const u32x4_t *)(a_base + (a_off[i] - qo) + (int64_t)k * 2) : zero;
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
    uint16_t *out = (uint16_t *)g.out;
    for (int it = tid; it < MF * (FUSED_UP ? 64 : 128); it += (int)blockDim.x) {
        const int l = it & 63, i = FUSED_UP ? it >> 6 : it >> 7, j = FUSED_UP ? 0 : (it >> 6) & 1;
        const int row = m0 + i * 16 + (l & 15), col = n0 + j * 16 + 4 * (l >> 4);
        if (row >= m_end || col >= g.N) continue;   // N is a multiple of 8
        float4 h = total(i, j, l);
        if (FUSED_UP) {
            const float4 u = total(i, 1, l);
            h.x = h.x * __frcp_rn(1.0f + __expf(-h.x)) * u.x;
            h.y = h.y * __frcp_rn(1.0f + __expf(-h.y)) * u.y;
            h.z = h.z * __frcp_rn(1.0f + __expf(-h.z)) * u.z;
            h.w = h.w * __frcp_rn(1.0f + __expf(-h.w)) * u.w;
        }
        *(uint2 *)(out + (int64_t)row * g.ldo + col) = make_uint2(pack_bf16x2(h.x, h.y), pack_bf16x2(h.z, h.w));
    }
}

// One workgroup per (segment, strip of weight rows): block = slot * n_strips + strip.  MF_MAX: fragments of 16
// rows that cover the launcher's bound on a segment's rows; a segment with fewer rows takes a shorter
// body, one with more is walked in pieces.
template <bool FUSED_UP, int MF_MAX>
__global__ __launch_bounds__(64 * MAX_WAVES) void gemm_bf16_stream_kernel(const GemmArgs g, int n_strips) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int slot = (int)blockIdx.x / n_strips, n0 = ((int)blockIdx.x - slot * n_strips) * Shape<FUSED_UP>::COLS;
    StaleRows stale;
    if (!FUSED_UP) stale = stale_rows(g);
    const int lo = __builtin_amdgcn_readfirstlane(g.seg_off ? g.seg_off[slot] : 0);
    const int hi = __builtin_amdgcn_readfirstlane(g.seg_off ? g.seg_off[slot + 1] : g.M_single);
    for (int m0 = lo; m0 < hi; m0 += MF_MAX * 16) {
        if (m0 > lo) __syncthreads();   // the sums of the rows before have been read
        const int m_end = min(hi, m0 + MF_MAX * 16), rows = m_end - m0;
        if (MF_MAX == 1 || rows <= 16) rows_body<FUSED_UP, 1>(g, slot, m0, m_end, n0, (float4 *)smem);
        else if (MF_MAX == 2 || rows <= 32) rows_body<FUSED_UP, MF_MAX < 2 ? MF_MAX : 2>(g, slot, m0, m_end, n0, (float4 *)smem);
        else if (rows <= 48) rows_body<FUSED_UP, MF_MAX < 3 ? MF_MAX : 3>(g, slot, m0, m_end, n0, (float4 *)smem);
        else rows_body<FUSED_UP, MF_MAX>(g, slot, m0, m_end, n0, (float4 *)smem);
    }
    if (FUSED_UP) share_record(g); else clear_stale_rows(g, stale);
}

}  // namespace strm
}  // namespace grace
