// The dispatch of the smallest batches by workgroups that do not wait for one another: every workgroup (one per token) does all of
// the index work from the logits, in LDS, and moves and writes what belongs to its token; workgroup 0 also writes the counts and
// offsets.  A launch of its own (route_permute.hip) or workgroups of the experts' gate+up projection (ffn_tiny.hip).
#pragma once
#include "bf16.h"
#include "common.h"
#include "gemm_common.h"
#include "route_device.h"
#include "wave_utils.h"

namespace grace {

inline bool tiny_batch(int T, int k, int E, int I) { return T >= 1 && T <= tiny_most_tokens(k, E, I); }

struct TinyArgs {
    const float *logits;
    int T, E, k, renorm;
    const uint32_t *rr_in;
    uint32_t *rr_out;
    const int32_t *cand_ptr, *cand_g;
    const uint32_t *cand_cum;
    int I, R, N;
    const int32_t *rank_ptr, *node_first_inst;
    int32_t *topk_expert;
    float *topk_weight;
    int32_t *topk_inst, *expert_count, *perm_pos, *perm_src, *inst_off, *rank_off, *node_off;
    const uint4 *x;
    int row_vec;
    uint4 *xp;
};
// (host) arguments of a checked call
inline TinyArgs tiny_args(const grace_table *table, int32_t local_rank, grace_policy policy, const float *logits, int32_t T, int32_t k,
                          int32_t renorm, const uint32_t *rr_in, uint32_t *rr_out, int32_t *topk_expert, float *topk_weight,
                          int32_t *topk_inst, int32_t *expert_count, const void *x, int32_t d, grace_dtype dt, int32_t *perm_pos,
                          int32_t *perm_src, int32_t *inst_off, int32_t *rank_off, int32_t *node_off, void *xp) {
    const int view = policy == GRACE_POLICY_WRR ? table->R : local_rank;
    return {logits, T, table->E, k, renorm, rr_in, rr_out, table->d_cand_ptr + (size_t)view * table->E, table->d_cand_g, table->d_cand_cum,
            table->I, table->R, table->N, table->d_rank_ptr, table->d_node_first_inst, topk_expert, topk_weight, topk_inst, expert_count,
            perm_pos, perm_src, inst_off, rank_off, node_off, (const uint4 *)x, x ? (int)((int64_t)d * (dt == GRACE_F32 ? 4 : 2) / 16) : 1,
            (uint4 *)xp};
}

struct TinyLds {
    uint16_t ecnt[TINY_MAX_ASG / 64][MAX_KEYS];   // requests per expert of 64 assignments, then before them
    uint16_t icnt[TINY_MAX_ASG / 64][MAX_KEYS];   // rows per instance of 64 assignments, then before them
    int16_t asg[TINY_MAX_ASG], inst[TINY_MAX_ASG], where[TINY_MAX_ASG];   // expert of every assignment, its instance, its position
    int16_t count[MAX_KEYS], only[MAX_KEYS];      // candidates of an expert; the first one
    uint32_t weight_sum[MAX_KEYS], rr[MAX_KEYS];
    int32_t ioff[MAX_KEYS + 1];
};

// How the gate takes the tokens.  WAVE: a wavefront per token, VPL experts per lane.  ROWS: a wavefront takes four (row_topk), 4 VPL
// experts per lane.  LANES: a lane takes a token, up to TINY_LANE_E experts.
enum class Gate { WAVE, ROWS, LANES };
constexpr int TINY_LANE_E = 16;

// Choices of all tokens by the workgroup: chosen(t, j, e) for choice j of token t.  PASSES: passes whose logits are in flight at a time;
// load(0), then choose().
template <int VPL, Gate GATE, int PASSES>
struct TinyGate {
    static_assert(GATE != Gate::LANES || VPL == 1, "up to 16 experts");
    static constexpr int NU = GATE == Gate::LANES ? TINY_LANE_E : GATE == Gate::ROWS ? 4 * VPL : VPL;   // experts per lane
    static constexpr int AT_ONCE = GATE == Gate::LANES ? 64 : GATE == Gate::ROWS ? 4 : 1;               // tokens per wavefront and pass
    const float *logits;
    int T, E, k, lane, wave, waves;
    float raw[PASSES][NU];

    __device__ __forceinline__ TinyGate(const float *logits, int T, int E, int k)
        : logits(logits), T(T), E(E), k(k), lane((int)threadIdx.x & 63), wave(__builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6)),
          waves((int)blockDim.x >> 6) {}
    __device__ __forceinline__ int token(int i) const {
        return (i * waves + wave) * AT_ONCE + (GATE == Gate::LANES ? lane : GATE == Gate::ROWS ? lane >> 4 : 0);
    }
    __device__ __forceinline__ void load(int i0) {
#pragma unroll
        for (int i = 0; i < PASSES; ++i)
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                const int t = token(i0 + i), e = GATE == Gate::LANES ? u : GATE == Gate::ROWS ? (lane & 15) + 16 * u : lane + 64 * u;
                raw[i][u] = (t < T && e < E) ? logits[(size_t)t * E + e] : -INFINITY;
            }
    }
    template <typename F>
    __device__ __forceinline__ void choose(F chosen) {
        for (int i0 = 0;;) {
#pragma unroll
            for (int i = 0; i < PASSES; ++i) {
                const int t = token(i0 + i);
                if (((i0 + i) * waves + wave) * AT_ONCE >= T) break;   // uniform per wavefront
#pragma unroll
                for (int u = 0; u < NU; ++u) raw[i][u] = not_all_ones(raw[i][u]);
                if constexpr (GATE == Gate::LANES) {
                    uint32_t key[NU];
#pragma unroll
                    for (int u = 0; u < NU; ++u) key[u] = u < E ? ordered_bits(raw[i][u] == 0.0f ? 0.0f : raw[i][u]) : 0u;
                    for (int j = 0; j < k; ++j) {   // the largest, equal ones by ascending id, leaves
                        uint32_t best = key[0];
                        int e = 0;
#pragma unroll
                        for (int u = 1; u < NU; ++u) {
                            const bool more = key[u] > best;
                            best = more ? key[u] : best;
                            e = more ? u : e;
                        }
                        if (t < T) chosen(t, j, e);   // (k is at most E: there is one)
#pragma unroll
                        for (int u = 0; u < NU; ++u) key[u] = e == u ? 0u : key[u];
                    }
                } else if constexpr (GATE == Gate::ROWS) {
                    row_topk<NU>(raw[i], lane & 15, E, k, [&](int j, int e) {
                        if (t < T && e < E) chosen(t, j, e);
                    });
                } else {
                    int rank[NU];
                    token_ranks<VPL, true>(raw[i], lane, E, k, rank);
#pragma unroll
                    for (int u = 0; u < NU; ++u)
                        if (lane + 64 * u < E && rank[u] < k) chosen(t, rank[u], lane + 64 * u);
                }
            }
            i0 += PASSES;
            if (i0 * waves * AT_ONCE >= T) break;
            load(i0);
        }
    }
};

// Bound by latency, so: candidates, the token's row and its logits are loaded ahead, and the gate weights, which only the caller needs, come
// last, under the row's stores.  PASSES: passes of the gate whose logits are in flight at a time.  ONE: a wavefront has 64 assignments at
// most and keeps what it knows of them in registers.  At least four wavefronts, a thread per expert and instance.  Workgroup `me` of
// args.T.
template <int VPL, Gate GATE, int PASSES, bool ONE>
__device__ __forceinline__ void tiny_dispatch(const TinyArgs &d, int me, TinyLds &s) {
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), threads = (int)blockDim.x, waves = threads >> 6;
    const int T = d.T, E = d.E, k = d.k, I = d.I, n = T * k, groups = (n + 63) >> 6;
    // ---- loads ahead: this wavefront's logits, the experts' candidates, the row to move
    TinyGate<VPL, GATE, PASSES> gate(d.logits, T, E, k);
    gate.load(0);
    const int e_own = min(tid, E - 1);
    const int cb = d.cand_ptr[e_own], ce = d.cand_ptr[e_own + 1];
    const uint32_t rr_own = d.rr_in ? d.rr_in[e_own] : 0u;
    const int copies = max(1, threads / d.row_vec), part = tid / d.row_vec, vec = tid - part * d.row_vec;   // `copies` groups of threads share the k rows
    uint4 row = make_uint4(0u, 0u, 0u, 0u);
    if (d.x && part < copies) row = d.x[(int64_t)me * d.row_vec + vec];
    float own[VPL];   // the last wavefront's: the token's logits, for its weights
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
        const int e = lane + 64 * v;
        own[v] = (wave == waves - 1 && e < E) ? d.logits[(size_t)me * E + e] : -INFINITY;
    }
    for (int i = tid; i < n; i += threads) s.asg[i] = -1;
    for (int g = wave; g < groups; g += waves)
        for (int i = lane; i < MAX_KEYS / 2; i += 64) {
            ((uint32_t *)s.ecnt[g])[i] = 0u;
            ((uint32_t *)s.icnt[g])[i] = 0u;
        }
    __syncthreads();
    const int only_own = d.cand_g[cb];
    const uint32_t sum_own = d.cand_cum[ce - 1];
    // ---- gate (the weights, which nothing here needs, at the end)
    gate.choose([&](int t, int j, int e) { s.asg[t * k + j] = (int16_t)e; });
    if (tid < E) {
        s.count[tid] = (int16_t)(ce - cb);
        s.only[tid] = (int16_t)only_own;
        s.weight_sum[tid] = sum_own;
        s.rr[tid] = rr_own;
    }
    __syncthreads();
    // ---- requests of each expert: in 64 assignments, before them, in all
    const uint64_t lt = lanemask_lt();
    const int ebits = bits_for(E), ibits = bits_for(I);
    int e_raw = -1, inst = 0;   // (ONE: of this lane's assignment, from here on; else of the one in hand)
    uint64_t same = 0;
    auto each = [&](auto f) {
        if constexpr (ONE) {
            if (wave < groups) f(wave, wave * 64 + lane);
        } else {
            for (int g = wave; g < groups; g += waves) f(g, g * 64 + lane);
        }
    };
    each([&](int g, int a) {
        e_raw = a < n ? s.asg[a] : -1;
        same = wave_match((uint32_t)max(e_raw, 0), e_raw >= 0, ebits);
        if (e_raw >= 0 && is_last_of(same)) s.ecnt[g][e_raw] = (uint16_t)__popcll(same);
    });
    __syncthreads();
    if (tid < E) {
        int32_t run = 0;
        for (int g = 0; g < groups; ++g) {
            const int32_t c = s.ecnt[g][tid];
            s.ecnt[g][tid] = (uint16_t)run;
            run += c;
        }
        if (me == 0) {
            d.expert_count[tid] = run;
            const uint64_t c = (uint64_t)s.rr[tid] + (uint64_t)(uint32_t)run;
            const uint32_t W = s.weight_sum[tid];
            if (d.rr_out) d.rr_out[tid] = (c >> 32) ? (uint32_t)(c % W) : (uint32_t)c % W;
        }
    }
    __syncthreads();
    // ---- replica pick; rows of each instance: in 64 assignments, before them, in all
    each([&](int g, int a) {
        if constexpr (!ONE) e_raw = a < n ? s.asg[a] : -1;
        const bool valid = e_raw >= 0;
        const int e = max(e_raw, 0);
        inst = valid ? s.only[e] : 0;
        const bool several = valid && s.count[e] > 1;
        if constexpr (!ONE) {
            if (__any(several)) same = wave_match((uint32_t)e, valid, ebits);
        }
        if (several) {
            const uint64_t c = (uint64_t)(uint32_t)s.ecnt[g][e] + (uint32_t)__popcll(same & lt) + (uint64_t)s.rr[e];
            inst = pick_candidate(c, e, d.cand_ptr, d.cand_g, d.cand_cum);
        }
        if (!ONE && a < n) s.inst[a] = (int16_t)inst;
        same = wave_match((uint32_t)inst, valid, ibits);
        if (valid && is_last_of(same)) s.icnt[g][inst] = (uint16_t)__popcll(same);
    });
    __syncthreads();
    if (tid < MAX_KEYS) {
        int32_t total = 0;
        for (int g = 0; g < groups; ++g) {
            const int32_t c = s.icnt[g][tid];
            s.icnt[g][tid] = (uint16_t)total;
            total += c;
        }
        s.ioff[tid] = total;
    }
    __syncthreads();
    if (wave == 0) {
        int32_t c[4], sum = 0;   // exclusive scan over the ids, four per lane
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            c[q] = s.ioff[lane * 4 + q];
            sum += c[q];
        }
        const int32_t incl = wave_scan_add(sum);
        int32_t run = incl - sum;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            s.ioff[lane * 4 + q] = run;
            run += c[q];
        }
        if (lane == 63) s.ioff[MAX_KEYS] = incl;
    }
    __syncthreads();
    // ---- positions, offsets, rows
    each([&](int g, int a) {
        if constexpr (!ONE) {
            e_raw = a < n ? s.asg[a] : -1;
            inst = a < n ? s.inst[a] : 0;
            same = wave_match((uint32_t)inst, e_raw >= 0, ibits);
        }
        if (a < n) {
            const bool valid = e_raw >= 0;
            const int pos = valid ? s.ioff[inst] + s.icnt[g][inst] + (int)__popcll(same & lt) : -1;
            s.where[a] = (int16_t)pos;
            if (a >= me * k && a < (me + 1) * k) {
                d.perm_pos[a] = pos;
                if (valid) {
                    d.topk_inst[a] = inst;
                    d.perm_src[pos] = a;
                }
            }
        }
    });
    if (me == 0) {
        for (int i = tid; i <= I; i += threads) d.inst_off[i] = s.ioff[i];
        for (int r = tid; r <= d.R; r += threads) d.rank_off[r] = s.ioff[d.rank_ptr[r]];
        for (int m = tid; m <= d.N; m += threads) d.node_off[m] = s.ioff[d.node_first_inst[m]];
    }
    __syncthreads();
    if (d.x && part < copies) {
        for (int v = vec; v < d.row_vec; v += threads) {   // more than once only if a row has more vectors than the workgroup threads
            if (v != vec) row = d.x[(int64_t)me * d.row_vec + v];
            for (int j = part; j < k; j += copies) {
                const int32_t p = s.where[me * k + j];
                if (p >= 0) nt_store16(row, &d.xp[(int64_t)p * d.row_vec + v]);
            }
        }
    }
    // ---- what the call returns of the token's gate
    if (wave == waves - 1) {
        int rank[VPL];
        float weight[VPL];
#pragma unroll
        for (int v = 0; v < VPL; ++v) rank[v] = k;
        for (int j = 0; j < k; ++j) {
            const int e_j = s.asg[me * k + j];
#pragma unroll
            for (int v = 0; v < VPL; ++v) rank[v] = e_j == lane + 64 * v ? j : rank[v];
        }
        token_weights<VPL>(own, lane, E, k, d.renorm, rank, weight);
#pragma unroll
        for (int v = 0; v < VPL; ++v)
            if (rank[v] < k) {
                d.topk_expert[(size_t)me * k + rank[v]] = lane + 64 * v;
                d.topk_weight[(size_t)me * k + rank[v]] = weight[v];
            }
    }
}

}  // namespace grace
