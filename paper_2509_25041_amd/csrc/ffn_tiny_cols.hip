// Gate+up projections of up to 8 tokens beside their dispatch (ffn_tiny.hip), dealt out evenly.
//
// A few tokens leave most slots of a rank without rows, and which ones is not known before the gate: with a workgroup per slot and strip most have
// nothing to do, and the others fall unevenly on the compute units.  Here every workgroup finds the rows of all slots from the logits (the
// gate of the dispatch, a few tokens per wavefront) and takes its share, one in as many as there are workgroups, of the units that these make: 4 output columns of a
// slot with rows.  Its wavefronts deal the parts of K of its units among themselves.
//
// Bound by latency (logits, gate and first weights 6 us), then by the weights.  Layer steps with cold weights, a workgroup per slot and strip -> dealt out,
// d = 2048, k = 8: one token, f = 1024, 64 experts 16.5 -> 15.5 us, 4 tokens 26.5 -> 23.9; f = 768, 128 experts, 8 tokens 25.6 -> 23.5; fp32, d
// = 1024, f = 704, k = 2, one token 17.3 -> 15.2.  For more than 8 tokens a second octet of activations takes too many loads' places (16 tokens of 128 experts
// 26.5 -> 27.9 us, of 64, f = 1024, 38.0 -> 36.0), also where the tokens wait in LDS.
#include <type_traits>

#include "ffn_tiny.h"
#include "gemm_stream.h"
#include "tiny_parts.h"

namespace grace {

struct ColsLds {
    uint32_t chose[MAX_KEYS];                // tokens (bits) that chose an expert
    int16_t slot[MAX_KEYS];                  // slots with rows
    int16_t rows[MAX_KEYS];
    uint8_t token[MAX_KEYS][TINY_COLS_T];    // of each row
    int segments;
};
constexpr int COLS_FIXED = (sizeof(ColsLds) + 15) / 16 * 16;

static_assert(TINY_COLS_T * GRACE_MAX_TOPK <= 64 * PART_WAVES, "a wavefront of the dispatch keeps 64 assignments");
constexpr int COLS_ITEMS = 64;   // partial sums of a round

// EL: bytes per element
template <int VPL, Gate GATE, int EL>
__global__ __launch_bounds__(PART_THREADS) void tiny_cols_kernel(const TinyUp a) {
    constexpr int DEPTH = 6;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const TinyArgs &d = a.dispatch;
    if ((int)blockIdx.x < d.T) {
        TinyLds &s = *(TinyLds *)smem;
        tiny_dispatch<VPL, GATE, GATE == Gate::WAVE ? 2 : 1, true>(d, (int)blockIdx.x, s);
        tiny_share_record(a, s);
        return;
    }
    ColsLds &s = *(ColsLds *)smem;
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), r = lane & 15, q = lane >> 4;
    const GemmArgs &g = a.up;
    float *const part = (float *)(smem + COLS_FIXED);   // [item][8 rows][4 of gate, 4 of up]
    // ---- rows of all slots
    TinyGate<VPL, GATE, GATE == Gate::WAVE ? 2 : 1> gate(d.logits, d.T, d.E, d.k);
    gate.load(0);
    const bool sorts = wave == PART_WAVES - 1;   // (the last one has the fewest tokens)
    uint4 span = make_uint4(0u, 0u, 0u, 1u);
    if (sorts && lane < g.S) span = a.slot_span[lane];
    if (tid < MAX_KEYS) s.chose[tid] = 0u;
    __syncthreads();
    gate.choose([&](int t, int, int e) { atomicOr(&s.chose[e], 1u << t); });
    uint32_t rr = sorts && a.several && d.rr_in && lane < g.S ? d.rr_in[span.x] : 0u;
    __syncthreads();
    if (sorts) {
        int count = 0;
        for (int s0 = 0; s0 < g.S; s0 += 64) {
            const int slot = s0 + lane;
            if (s0 > 0 && slot < g.S) {
                span = a.slot_span[slot];
                rr = a.several && d.rr_in ? d.rr_in[span.x] : 0u;
            }
            uint32_t mask = slot < g.S ? s.chose[span.x] : 0u, mine = mask;
            if (a.several) {   // request number -> instance: this one's if the number falls into its interval
                mine = 0u;
                uint32_t number = rr % span.w;
                for (; mask; mask &= mask - 1) {
                    mine |= number >= span.y && number < span.z ? mask & (0u - mask) : 0u;
                    number = number + 1 == span.w ? 0u : number + 1;
                }
            }
            const uint64_t hit = __ballot(mine != 0u);
            const int at = count + (int)__popcll(hit & lanemask_lt());
            if (mine) {
                s.slot[at] = (int16_t)slot;
                s.rows[at] = (int16_t)__popc(mine);
                for (int i = 0; mine; mine &= mine - 1) s.token[at][i++] = (uint8_t)(__ffs(mine) - 1);
            }
            count += (int)__popcll(hit);
        }
        if (lane == 0) s.segments = count;
    }
    __syncthreads();
    // ---- this workgroup's units; neighbouring ones on one XCD, whose L2 makes whole lines of their stores
    const int hit = __builtin_amdgcn_readfirstlane(s.segments), groups = g.N >> 2, total = hit * groups;
    const int b = (int)blockIdx.x - d.T, blocks = (int)gridDim.x - d.T, me = (b & 7) * (blocks >> 3) + (b >> 3);   // (blocks is a multiple of 8)
    const int row_bytes = g.K * EL, steps = row_bytes >> 7;
    const auto a_rsrc = rsrc_of((const char *)g.A);
    // rows 0 to 3 and 8 to 11 of a fragment: the two halves of a step of the gate's rows, the others the up projection's
    const int64_t b_lane = (int64_t)(r & 3) * row_bytes + (r >> 3) * 64 + q * 16;
    for (int u0 = me; u0 < total; u0 += COLS_ITEMS * blocks) {
        if (u0 != me) __syncthreads();   // the sums before have been read
        const int units = min(COLS_ITEMS, (total - u0 + blocks - 1) / blocks);
        const int parts_log = parts_log_of(units, steps), parts = 1 << parts_log, items = units << parts_log;
        uint32_t a_off;
        const char *from;
        walk_parts<EL, 1, DEPTH, true>(
            wave, items, parts_log, steps,
            [&](int i) {
                const int u = u0 + i * blocks, seg = u / groups, n0 = (u - seg * groups) * 4;
                const int slot = __builtin_amdgcn_readfirstlane((int)s.slot[seg]), row = min(r & 7, s.rows[seg] - 1);
                a_off = (uint32_t)s.token[seg][row] * (uint32_t)row_bytes + (uint32_t)(r >> 3) * 64u + (uint32_t)q * 16u;
                from = ((r >> 2) & 1 ? (const char *)g.B1 : (const char *)g.B0) + (int64_t)slot * g.b_slot_stride * EL + (int64_t)n0 * row_bytes + b_lane;
            },
            [&](int at, u32x4_t (&rb)[1], u32x4_t (&ra)[1]) {
                rb[0] = *(const u32x4_t *)(from + at);
                ra[0] = load16(a_rsrc, a_off, (uint32_t)at);
            },
            [&](int item, int, const f32x4_t &sum) {
                if (q < 2 && r < 8) *(f32x4_t *)&part[(item * 8 + r) * 8 + 4 * q] = sum;
            });
        __syncthreads();
        // sums in the order of the parts, activation, four columns per thread
        for (int i = tid; i < units * 8; i += PART_THREADS) {
            const int u = u0 + (i >> 3) * blocks, seg = u / groups, row = i & 7, col = (u - seg * groups) * 4;
            if (row >= s.rows[seg]) continue;
            f32x4_t h = {0.0f, 0.0f, 0.0f, 0.0f}, up = h;
            for (int p = 0; p < parts; ++p) {
                const float *const at = &part[((((i >> 3) << parts_log) + p) * 8 + row) * 8];
                h += *(const f32x4_t *)at;
                up += *(const f32x4_t *)(at + 4);
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) h[c] = (EL == 2 ? h[c] * __frcp_rn(1.0f + __expf(-h[c])) : h[c] / (1.0f + expf(-h[c]))) * up[c];
            const int64_t o = ((int64_t)s.slot[seg] * d.T + row) * g.ldo + col;
            if constexpr (EL == 2) *(uint2 *)((uint16_t *)g.out + o) = make_uint2(pack_bf16x2(h[0], h[1]), pack_bf16x2(h[2], h[3]));
            else *(float4 *)((float *)g.out + o) = make_float4(h[0], h[1], h[2], h[3]);
        }
    }
}

constexpr int COLS_LDS = std::max((int)sizeof(TinyLds), COLS_FIXED + COLS_ITEMS * 8 * 8 * 4);
const void *tiny_cols_kernel_of(grace_dtype dt, int T, int E) {
    using std::integral_constant;
    auto by_gate = [&](auto vpl, auto gate) {
        constexpr int VPL = decltype(vpl)::value;
        constexpr Gate GATE = decltype(gate)::value;
        return dt == GRACE_BF16 ? (const void *)tiny_cols_kernel<VPL, GATE, 2> : (const void *)tiny_cols_kernel<VPL, GATE, 4>;
    };
    if (E > 128) return by_gate(integral_constant<int, 4>{}, integral_constant<Gate, Gate::WAVE>{});
    if (E > 64) return by_gate(integral_constant<int, 2>{}, integral_constant<Gate, Gate::WAVE>{});
    if (T <= 4) return by_gate(integral_constant<int, 1>{}, integral_constant<Gate, Gate::WAVE>{});
    if (E <= TINY_LANE_E) return by_gate(integral_constant<int, 1>{}, integral_constant<Gate, Gate::LANES>{});
    return by_gate(integral_constant<int, 1>{}, integral_constant<Gate, Gate::ROWS>{});
}
void launch_tiny_cols(const TinyUp &a, grace_dtype dt, int n_cu, hipStream_t st) {
    TinyUp args = a;
    void *params[] = {&args};
    const TinyArgs &d = a.dispatch;
    (void)hipLaunchKernel(tiny_cols_kernel_of(dt, d.T, d.E), dim3((unsigned)(d.T + (n_cu + 7) / 8 * 8)), dim3(PART_THREADS), params, COLS_LDS, st);
}

}  // namespace grace
