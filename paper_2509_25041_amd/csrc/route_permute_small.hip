// grace_route_permute: grace_route followed by grace_permute as one call.
//
// Any batch: the replica pick also counts its choices per permutation chunk and
// instance (into counters the top-k kernel cleared), so the permutation's own
// histogram launch is dropped: top-k, pick, positions, row scatter.
//
// Decode-sized batches (a few hundred tokens) are bound by launch latency: the
// two calls need five launches of kernels that each run a few microseconds.  When
// the batch is small enough, the top-k gate (one wavefront per token, spread over
// the device) is followed by ONE single-workgroup kernel that does all the index
// work, every wavefront owning a contiguous range of assignments:
//   1. request counters    scan of the per-wavefront expert counts (Section 4.3)
//   2. replica pick        Algorithm 4 tier + weighted round-robin, per wavefront in order
//   3. offsets             per instance / rank / node, scan of the per-wavefront instance counts
//   4. positions           stable rank of every assignment in (node, rank, slot) order (Section 5)
// and by the row scatter: three launches.  Still smaller ones take a single launch (route_permute_tiny_kernel).
// Outputs are identical either way (all integer work is exact and order-independent).
#include <mutex>
#include <type_traits>

#include "bf16.h"
#include "common.h"
#include "route_device.h"
#include "stable_sort.h"
#include "wave_utils.h"

namespace grace {

constexpr int SMALL_THREADS = 1024, SMALL_WAVES = SMALL_THREADS / 64;
constexpr int SMALL_MAX_KEYS = 256;      // experts and instances the LDS tables hold
constexpr int SMALL_MAX_PER_WAVE = 256;  // assignments one wavefront walks

inline bool small_batch(int T, int k, int E, int I) {
    return T >= 1 && E <= SMALL_MAX_KEYS && I <= SMALL_MAX_KEYS &&
           ceil_div(T, SMALL_WAVES) * k <= SMALL_MAX_PER_WAVE;
}

// Bound by latency: a lane's assignments (four at most) are loaded at once and stay in registers, and the candidates of every
// expert are loaded ahead of the loops, which have no global load left but those of experts with several candidates (a chain
// of three per group of 64 assignments before: 512 tokens, k = 8 15.1 -> 11.4 us, 1000 tokens, k = 2 9.5 -> 7.5 us).
__global__ __launch_bounds__(SMALL_THREADS) void dispatch_small_kernel(
    int T, int E, int k, const uint32_t *__restrict__ rr_in, uint32_t *__restrict__ rr_out,
    const int32_t *__restrict__ cand_ptr, const int32_t *__restrict__ cand_g, const uint32_t *__restrict__ cand_cum, int I,
    int R, int N, const int32_t *__restrict__ rank_ptr, const int32_t *__restrict__ node_first_inst,
    const int32_t *__restrict__ topk_expert, int32_t *__restrict__ topk_inst, int32_t *__restrict__ expert_count,
    int32_t *__restrict__ perm_pos, int32_t *__restrict__ perm_src, int32_t *__restrict__ inst_off,
    int32_t *__restrict__ rank_off, int32_t *__restrict__ node_off) {
    constexpr int GROUPS = SMALL_MAX_PER_WAVE / 64;
    __shared__ int32_t ecnt[SMALL_WAVES][SMALL_MAX_KEYS];  // requests per expert of a wavefront, then before it
    __shared__ int32_t icnt[SMALL_WAVES][SMALL_MAX_KEYS];  // rows per instance of a wavefront, then before it
    __shared__ int32_t count[SMALL_MAX_KEYS], only[SMALL_MAX_KEYS];   // candidates of an expert; the first one
    __shared__ uint32_t rr[SMALL_MAX_KEYS];
    __shared__ int32_t ioff[SMALL_MAX_KEYS + 1];
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int tpw = (T + SMALL_WAVES - 1) / SMALL_WAVES;  // tokens per wavefront
    const int t0 = min(T, wave * tpw), t1 = min(T, t0 + tpw);
    const int n_w = (t1 - t0) * k;                         // assignments of this wavefront, in order
    const int64_t a0 = (int64_t)t0 * k;
    int key[GROUPS];   // expert, then instance, of this lane's assignments; -1: none, or an expert id outside the table
#pragma unroll
    for (int q = 0; q < GROUPS; ++q) key[q] = q * 64 + lane < n_w ? topk_expert[a0 + q * 64 + lane] : -1;
    const int e_own = min(tid, E - 1);
    const int cb = cand_ptr[e_own], ce = cand_ptr[e_own + 1];
    const uint32_t rr_own = rr_in ? rr_in[e_own] : 0u;
    for (int i = lane; i < SMALL_MAX_KEYS; i += 64) {
        ecnt[wave][i] = 0;
        icnt[wave][i] = 0;
    }
    const int ebits = bits_for(E), ibits = bits_for(I);
    const uint64_t lt = lanemask_lt();
    // The LDS operations of one wavefront execute in program order, so a counter updated by the last
    // lane of a match set is seen by the next group of 64 assignments.
    // ---- 0. this wavefront's experts and their counts ---------------------------------------------
#pragma unroll
    for (int q = 0; q < GROUPS; ++q) {
        if (q * 64 >= n_w) break;   // uniform per wavefront
        if ((unsigned)key[q] >= (unsigned)E) key[q] = -1;
        const bool valid = key[q] >= 0;
        const int e = valid ? key[q] : 0;
        const uint64_t same = wave_match((uint32_t)e, valid, ebits);
        if (valid && is_last_of(same)) wave_ctr_add(&ecnt[wave][e], (int32_t)__popcll(same));
        wave_ctr_fence();
    }
    const uint32_t weight_sum = cand_cum[ce - 1];
    if (tid < E) {
        count[tid] = ce - cb;
        only[tid] = cand_g[cb];
        rr[tid] = rr_own;
    }
    __syncthreads();
    // ---- 1. requests of each expert before each wavefront; totals -----------------------------
    if (tid < E) {
        int32_t run = 0;
#pragma unroll
        for (int w = 0; w < SMALL_WAVES; ++w) {
            const int32_t c = ecnt[w][tid];
            ecnt[w][tid] = run;
            run += c;
        }
        expert_count[tid] = run;
        const uint64_t c = (uint64_t)rr_own + (uint64_t)(uint32_t)run;
        if (rr_out) rr_out[tid] = (c >> 32) ? (uint32_t)(c % weight_sum) : (uint32_t)c % weight_sum;
    }
    __syncthreads();
    // ---- 2. replica pick, in assignment order; instance counts ---------------------------------
#pragma unroll
    for (int q = 0; q < GROUPS; ++q) {
        if (q * 64 >= n_w) break;
        const bool valid = key[q] >= 0;
        const int e = valid ? key[q] : 0;
        const uint64_t same = wave_match((uint32_t)e, valid, ebits);
        int g = 0;
        if (valid) {
            g = only[e];
            if (count[e] > 1) {
                const uint64_t c = (uint64_t)(uint32_t)wave_ctr_load(&ecnt[wave][e]) + (uint32_t)__popcll(same & lt) + (uint64_t)rr[e];
                g = pick_candidate(c, e, cand_ptr, cand_g, cand_cum);
            }
            topk_inst[a0 + q * 64 + lane] = g;
            key[q] = g;
        }
        if (valid && is_last_of(same)) wave_ctr_add(&ecnt[wave][e], (int32_t)__popcll(same));
        const uint64_t same_g = wave_match((uint32_t)g, valid, ibits);
        if (valid && is_last_of(same_g)) wave_ctr_add(&icnt[wave][g], (int32_t)__popcll(same_g));
        wave_ctr_fence();
    }
    __syncthreads();
    // ---- 3. rows of each instance before each wavefront; offsets --------------------------------
    int32_t total = 0;
    if (tid < I) {
#pragma unroll
        for (int w = 0; w < SMALL_WAVES; ++w) {
            const int32_t c = icnt[w][tid];
            icnt[w][tid] = total;
            total += c;
        }
    }
    if (tid < SMALL_MAX_KEYS) ioff[tid] = total;  // totals, scanned below (zero for ids >= I)
    __syncthreads();
    if (wave == 0) {
        // exclusive scan over the ids: each lane owns four consecutive ids
        int32_t c[4], s = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            c[q] = ioff[lane * 4 + q];
            s += c[q];
        }
        const int32_t incl = wave_scan_add(s);
        int32_t run = incl - s;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            ioff[lane * 4 + q] = run;
            run += c[q];
        }
        if (lane == 63) ioff[SMALL_MAX_KEYS] = incl;  // grand total = offset of every id >= I
    }
    __syncthreads();
    for (int i = tid; i <= I; i += SMALL_THREADS) inst_off[i] = ioff[i];
    for (int r = tid; r <= R; r += SMALL_THREADS) rank_off[r] = ioff[rank_ptr[r]];
    for (int n = tid; n <= N; n += SMALL_THREADS) node_off[n] = ioff[node_first_inst[n]];
    // ---- 4. positions ---------------------------------------------------------------------------
#pragma unroll
    for (int q = 0; q < GROUPS; ++q) {
        if (q * 64 >= n_w) break;
        const int64_t a = a0 + q * 64 + lane;
        const bool valid = key[q] >= 0;
        const int g = valid ? key[q] : 0;
        const uint64_t same = wave_match((uint32_t)g, valid, ibits);
        if (valid) {
            const int32_t pos = ioff[g] + wave_ctr_load(&icnt[wave][g]) + (int32_t)__popcll(same & lt);
            perm_pos[a] = pos;
            perm_src[pos] = (int32_t)a;
        } else if (q * 64 + lane < n_w) {
            perm_pos[a] = -1;  // expert id outside the table: no row
        }
        if (valid && is_last_of(same)) wave_ctr_add(&icnt[wave][g], (int32_t)__popcll(same));
        wave_ctr_fence();
    }
}

// The smallest batches: top-k, index work and row movement in one launch.  Three launches of 2 to 7 us each wait for one
// another's first loads there, while all the index work of 64 tokens is a few microseconds for one workgroup.  So every
// workgroup (one per token) does all of it from the logits, in LDS, and moves and writes what belongs to its token; workgroup 0 also
// writes the counts and offsets.  Bound by latency, so: a wavefront takes a token in the gate, or four (row_topk) past 16 tokens,
// and at most 64 assignments afterwards (each lane keeps its own in registers); candidates, the token's row and its logits
// are loaded ahead; the gate weights, which only the caller needs, come last, under the row's stores.
// Layer steps, the three launches -> this one (1, 16, 64 tokens): 64 experts, k = 8 24.3 -> 20.8, 30.6 -> 25.0, 38.0 -> 33.9 us; 8 experts, k = 2
// 22.8 -> 17.8, 30.8 -> 27.2, 34.9 -> 30.5 us; 128 experts, k = 8 22.8 -> 18.8, 31.1 -> 24.0 us.  Where the line lies: every workgroup
// repeats the gate of all tokens, so the call (replayed from a graph) gains less with each.  96 tokens, 64 experts, k = 3, 4, 5, 6, 8: three
// launches as the next larger batch takes them 10.4, 10.4, 11.0, 11.2, 11.8, this one 7.5, 8.2, 8.6, 9.4, 10.5 us; 85 tokens, k = 12 is the most
// assignments.  Past 96 tokens k = 6 and 8 are about even in a step (128 tokens 56.7 -> 57.6, 39.1 -> 38.3 us).  256 tokens with k = 1, 2, where four
// passes of the wavefronts end: 9.1, 10.0 to 10.6 against 10.9, 10.4 to 11.0 us.  128 and 256 experts, 32 tokens, k = 8, two passes: 9.5 and 11.4
// against 12.3 and 14.0 us (33 tokens); four tokens by rows there 33 tokens 32.1 -> 32.2, 64 tokens 34.9 -> 36.1 us a step.
constexpr int TINY_MAX_ASG = 1024, TINY_MAX_WAVES = 16;
constexpr int TINY_MAX_T = 6 * TINY_MAX_WAVES, TINY_MAX_T_TOP2 = 16 * TINY_MAX_WAVES, TINY_MAX_T_WIDE = 2 * TINY_MAX_WAVES;
inline bool tiny_batch(int T, int k, int E, int I) {
    return T >= 1 && T <= (E > 64 ? TINY_MAX_T_WIDE : k > 2 ? TINY_MAX_T : TINY_MAX_T_TOP2) && (int64_t)T * k <= TINY_MAX_ASG && E <= SMALL_MAX_KEYS &&
           I <= SMALL_MAX_KEYS;
}

// VPL: experts per lane where a wavefront takes a token; ROWS: a wavefront takes four tokens at a time.  PASSES: how often.
template <int VPL, bool ROWS, int PASSES>
__global__ __launch_bounds__(64 * TINY_MAX_WAVES) void route_permute_tiny_kernel(
    const float *__restrict__ logits, int T, int E, int k, int renorm, const uint32_t *__restrict__ rr_in,
    uint32_t *__restrict__ rr_out, const int32_t *__restrict__ cand_ptr, const int32_t *__restrict__ cand_g,
    const uint32_t *__restrict__ cand_cum, int I, int R, int N, const int32_t *__restrict__ rank_ptr,
    const int32_t *__restrict__ node_first_inst, int32_t *__restrict__ topk_expert, float *__restrict__ topk_weight,
    int32_t *__restrict__ topk_inst, int32_t *__restrict__ expert_count, int32_t *__restrict__ perm_pos,
    int32_t *__restrict__ perm_src, int32_t *__restrict__ inst_off, int32_t *__restrict__ rank_off,
    int32_t *__restrict__ node_off, const uint4 *__restrict__ x, int row_vec, uint4 *__restrict__ xp) {
    __shared__ int32_t ecnt[TINY_MAX_WAVES][SMALL_MAX_KEYS];   // requests per expert of a wavefront, then before it
    __shared__ int32_t icnt[TINY_MAX_WAVES][SMALL_MAX_KEYS];   // rows per instance of a wavefront, then before it
    __shared__ int32_t asg[TINY_MAX_ASG], where[TINY_MAX_ASG]; // expert of every assignment; its position
    __shared__ int32_t count[SMALL_MAX_KEYS], only[SMALL_MAX_KEYS];   // candidates of an expert; the first one
    __shared__ uint32_t weight_sum[SMALL_MAX_KEYS], rr[SMALL_MAX_KEYS];
    __shared__ int32_t ioff[SMALL_MAX_KEYS + 1];
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6, threads = (int)blockDim.x, waves = threads >> 6;
    const int n = T * k, groups = (n + 63) >> 6, me = (int)blockIdx.x;   // groups <= waves; a workgroup per token
    // ---- loads ahead: this wavefront's logits, the experts' candidates, the row to move
    static_assert(!ROWS || VPL == 1, "row_topk takes up to 64 experts");
    constexpr int NU = ROWS ? 4 : VPL;   // experts per lane
    const int r = ROWS ? lane & 15 : lane;
    float raw[PASSES][NU];
    auto token = [&](int i) { return ROWS ? (i * waves + wave) * 4 + (lane >> 4) : i * waves + wave; };
#pragma unroll
    for (int i = 0; i < PASSES; ++i)
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int t = token(i), e = r + (ROWS ? 16 : 64) * u;
            raw[i][u] = (t < T && e < E) ? logits[(size_t)t * E + e] : -INFINITY;
        }
    const int e_own = min(tid, E - 1);
    const int cb = cand_ptr[e_own], ce = cand_ptr[e_own + 1];
    const uint32_t rr_own = rr_in ? rr_in[e_own] : 0u;
    const int copies = max(1, threads / row_vec), part = tid / row_vec, vec = tid - part * row_vec;   // `copies` groups of threads share the k rows
    uint4 row = make_uint4(0u, 0u, 0u, 0u);
    if (x && part < copies) row = x[(int64_t)me * row_vec + vec];
    float own[VPL];   // the last wavefront's: the token's logits, for its weights
#pragma unroll
    for (int v = 0; v < VPL; ++v) {
        const int e = lane + 64 * v;
        own[v] = (wave == waves - 1 && e < E) ? logits[(size_t)me * E + e] : -INFINITY;
    }
    for (int i = tid; i < n; i += threads) asg[i] = -1;
    for (int i = lane; i < SMALL_MAX_KEYS; i += 64) {
        ecnt[wave][i] = 0;
        icnt[wave][i] = 0;
    }
    __syncthreads();
    // ---- gate (the weights, which nothing here needs, at the end)
#pragma unroll
    for (int i = 0; i < PASSES; ++i) {
        const int t = token(i);
        if ((ROWS ? (i * waves + wave) * 4 : t) >= T) break;   // uniform per wavefront
        if constexpr (ROWS) {
            row_topk(raw[i], r, E, k, [&](int j, int e) {
                if (t < T && e < E) asg[t * k + j] = e;
            });
        } else {
            int rank[NU];
            token_ranks<VPL, true>(raw[i], lane, E, k, rank);
#pragma unroll
            for (int u = 0; u < NU; ++u)
                if (lane + 64 * u < E && rank[u] < k) asg[t * k + rank[u]] = lane + 64 * u;
        }
    }
    if (tid < E) {
        count[tid] = ce - cb;
        only[tid] = cand_g[cb];
        weight_sum[tid] = cand_cum[ce - 1];
        rr[tid] = rr_own;
    }
    __syncthreads();
    // ---- requests of each expert: in the group, before it, in all
    const uint64_t lt = lanemask_lt();
    const int a = wave * 64 + lane;
    int e = a < n ? asg[a] : -1;
    const bool valid = e >= 0;
    if (!valid) e = 0;
    uint64_t same = 0;
    if (wave < groups) {
        same = wave_match((uint32_t)e, valid, bits_for(E));
        if (valid && is_last_of(same)) ecnt[wave][e] = (int32_t)__popcll(same);
    }
    __syncthreads();
    if (tid < E) {
        int32_t run = 0;
        for (int w = 0; w < groups; ++w) {
            const int32_t c = ecnt[w][tid];
            ecnt[w][tid] = run;
            run += c;
        }
        if (me == 0) {
            expert_count[tid] = run;
            const uint64_t c = (uint64_t)rr[tid] + (uint64_t)(uint32_t)run;
            const uint32_t W = weight_sum[tid];
            if (rr_out) rr_out[tid] = (c >> 32) ? (uint32_t)(c % W) : (uint32_t)c % W;
        }
    }
    __syncthreads();
    // ---- replica pick; rows of each instance: in the group, before it, in all
    int g = 0;
    if (valid) {
        if (count[e] == 1) {
            g = only[e];
        } else {
            const uint64_t c = (uint64_t)(uint32_t)ecnt[wave][e] + (uint32_t)__popcll(same & lt) + (uint64_t)rr[e];
            g = pick_candidate(c, e, cand_ptr, cand_g, cand_cum);
        }
    }
    if (wave < groups) {
        same = wave_match((uint32_t)g, valid, bits_for(I));
        if (valid && is_last_of(same)) icnt[wave][g] = (int32_t)__popcll(same);
    }
    __syncthreads();
    if (tid < SMALL_MAX_KEYS) {
        int32_t total = 0;
        for (int w = 0; w < groups; ++w) {
            const int32_t c = icnt[w][tid];
            icnt[w][tid] = total;
            total += c;
        }
        ioff[tid] = total;
    }
    __syncthreads();
    if (wave == 0) {
        int32_t c[4], s = 0;   // exclusive scan over the ids, four per lane
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            c[q] = ioff[lane * 4 + q];
            s += c[q];
        }
        const int32_t incl = wave_scan_add(s);
        int32_t run = incl - s;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            ioff[lane * 4 + q] = run;
            run += c[q];
        }
        if (lane == 63) ioff[SMALL_MAX_KEYS] = incl;
    }
    __syncthreads();
    // ---- positions, offsets, rows
    if (a < n) {
        const int pos = valid ? ioff[g] + icnt[wave][g] + (int32_t)__popcll(same & lt) : -1;
        where[a] = pos;
        if (a >= me * k && a < (me + 1) * k) {
            perm_pos[a] = pos;
            if (valid) {
                topk_inst[a] = g;
                perm_src[pos] = a;
            }
        }
    }
    if (me == 0) {
        for (int i = tid; i <= I; i += threads) inst_off[i] = ioff[i];
        for (int r = tid; r <= R; r += threads) rank_off[r] = ioff[rank_ptr[r]];
        for (int m = tid; m <= N; m += threads) node_off[m] = ioff[node_first_inst[m]];
    }
    __syncthreads();
    if (x && part < copies) {
        for (int v = vec; v < row_vec; v += threads) {   // more than once only if a row has more vectors than the workgroup threads
            if (v != vec) row = x[(int64_t)me * row_vec + v];
            for (int j = part; j < k; j += copies) {
                const int32_t p = where[me * k + j];
                if (p >= 0) nt_store16(row, &xp[(int64_t)p * row_vec + v]);
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
            const int e_j = asg[me * k + j];
#pragma unroll
            for (int v = 0; v < VPL; ++v) rank[v] = e_j == lane + 64 * v ? j : rank[v];
        }
        token_weights<VPL>(own, lane, E, k, renorm, rank, weight);
#pragma unroll
        for (int v = 0; v < VPL; ++v)
            if (rank[v] < k) {
                topk_expert[(size_t)me * k + rank[v]] = lane + 64 * v;
                topk_weight[(size_t)me * k + rank[v]] = weight[v];
            }
    }
}

}  // namespace grace

using namespace grace;

static int route_permute_impl(const grace_table *table, int32_t local_rank, grace_policy policy, const float *logits,
                             int32_t T, int32_t E, int32_t k, int32_t renorm, const uint32_t *rr_in, uint32_t *rr_out,
                             int32_t *topk_expert, float *topk_weight, int32_t *topk_inst, int32_t *expert_count,
                             const void *x, int32_t d, grace_dtype dt, int32_t *perm_pos, int32_t *perm_src,
                             int32_t *inst_off, int32_t *rank_off, int32_t *node_off, void *xp, void *ws, void *stream) {
    hipStream_t st = (hipStream_t)stream;
    int rc;
    // the shared-histogram path counts with 32-bit indices; sizes beyond that take the two calls
    const bool hist_fits = ceil_div((int64_t)T * k, PERM_CHUNK) * table->I <= (int64_t)1 << 30;
    if (T == 0 || !hist_fits) {
        rc = grace_route(table, local_rank, policy, logits, T, E, k, renorm, rr_in, rr_out, topk_expert, topk_weight,
                         topk_inst, expert_count, ws, stream);
        if (rc != GRACE_OK) return rc;
        return grace_permute(table, topk_inst, T, k, x, d, dt, perm_pos, perm_src, inst_off, rank_off, node_off, xp, ws,
                             stream);
    }
    if (!small_batch(T, k, E, table->I)) {
        const int I = table->I;
        const int64_t n = (int64_t)T * k;
        const int nchunks = (int)ceil_div(n, PERM_CHUNK);
        int32_t *phist = (int32_t *)((char *)ws + fused_perm_ws_offset(T, E));
        int32_t *pbase = (int32_t *)((char *)phist + align_up((size_t)nchunks * I * 4, 256));
        rc = launch_route(table, local_rank, policy, logits, T, E, k, renorm, rr_in, rr_out, topk_expert, topk_weight,
                          topk_inst, expert_count, ws, phist, st);
        if (rc != GRACE_OK) return rc;
        const char *failed = stable_sort_launch(table, topk_inst, n, I, 1, phist, pbase, table->R, table->N, table->d_rank_ptr,
                                                table->d_node_first_inst, inst_off, rank_off, node_off, perm_pos, perm_src,
                                                st, /*hist_ready=*/true);
        if (failed) return fail(GRACE_EHIP, "route_permute: launch of %s failed", failed);
        if (x) return launch_scatter_rows(x, T, k, d, dt, perm_pos, xp, st);
        return GRACE_OK;
    }
    const int32_t *cand_ptr = table->d_cand_ptr + (size_t)(policy == GRACE_POLICY_WRR ? table->R : local_rank) * E;
    if (tiny_batch(T, k, E, table->I)) {
        const int row_vec = x ? (int)((int64_t)d * (dt == GRACE_F32 ? 4 : 2) / 16) : 1;
        int waves = 4;   // a thread per expert and instance, a wavefront per 64 assignments and, up to the most, per token or four
        const bool rows = E <= 64 && T > TINY_MAX_WAVES;
        while (waves < TINY_MAX_WAVES && waves * (rows ? 4 : 1) < T) waves *= 2;
        while (waves * 64 < T * k) waves *= 2;
        auto launch = [&](auto vpl) {
            constexpr int VPL = decltype(vpl)::value;
            auto *kern = route_permute_tiny_kernel<VPL, false, 1>;
            if constexpr (VPL == 1) {
                if (rows) kern = T <= 4 * waves ? route_permute_tiny_kernel<1, true, 1> : T <= 8 * waves ? route_permute_tiny_kernel<1, true, 2>
                                                                                                : route_permute_tiny_kernel<1, true, 4>;
            } else if (T > waves) {
                kern = route_permute_tiny_kernel<VPL, false, 2>;
            }
            kern<<<T, waves * 64, 0, st>>>(
                logits, T, E, k, renorm, rr_in, rr_out, cand_ptr, table->d_cand_g, table->d_cand_cum, table->I, table->R, table->N,
                table->d_rank_ptr, table->d_node_first_inst, topk_expert, topk_weight, topk_inst, expert_count, perm_pos, perm_src,
                inst_off, rank_off, node_off, (const uint4 *)x, row_vec, (uint4 *)xp);
        };
        if (E <= 64) launch(std::integral_constant<int, 1>{});
        else if (E <= 128) launch(std::integral_constant<int, 2>{});
        else if (E <= 192) launch(std::integral_constant<int, 3>{});
        else launch(std::integral_constant<int, 4>{});
        GRACE_LAUNCH_CHECK("route_permute_tiny_kernel");
        return GRACE_OK;
    }
    rc = launch_topk(logits, T, E, k, renorm, topk_expert, topk_weight, (int32_t *)ws, nullptr, 0, st);
    if (rc != GRACE_OK) return rc;
    dispatch_small_kernel<<<1, SMALL_THREADS, 0, st>>>(T, E, k, rr_in, rr_out, cand_ptr, table->d_cand_g, table->d_cand_cum,
                                                      table->I, table->R, table->N, table->d_rank_ptr,
                                                      table->d_node_first_inst, topk_expert, topk_inst, expert_count,
                                                      perm_pos, perm_src, inst_off, rank_off, node_off);
    GRACE_LAUNCH_CHECK("dispatch_small_kernel");
    if (x) return launch_scatter_rows(x, T, k, d, dt, perm_pos, xp, st);
    return GRACE_OK;
}

extern "C" int grace_route_permute(const grace_table *table, int32_t local_rank, grace_policy policy, const float *logits,
                                   int32_t T, int32_t E, int32_t k, int32_t renorm, const uint32_t *rr_in,
                                   uint32_t *rr_out, int32_t *topk_expert, float *topk_weight, int32_t *topk_inst,
                                   int32_t *expert_count, const void *x, int32_t d, grace_dtype dt, int32_t *perm_pos,
                                   int32_t *perm_src, int32_t *inst_off, int32_t *rank_off, int32_t *node_off, void *xp,
                                   void *ws, void *stream) {
    int rc = check_route_args(table, local_rank, policy, logits, T, E, k, rr_in, rr_out, topk_expert, topk_weight, topk_inst,
                              expert_count, ws);
    if (rc != GRACE_OK) return rc;
    rc = check_permute_args(table, topk_inst, T, k, x, d, dt, perm_pos, perm_src, inst_off, rank_off, node_off, xp, ws);
    if (rc != GRACE_OK) return rc;
    return route_permute_impl(table, local_rank, policy, logits, T, E, k, renorm, rr_in, rr_out, topk_expert, topk_weight,
                              topk_inst, expert_count, x, d, dt, perm_pos, perm_src, inst_off, rank_off, node_off, xp, ws,
                              stream);
}

// ---- the same call for callers that cannot allocate ------------------------------------------------
// The index kernels' scratch (chunk histograms and their prefix sums) lives in a file-scope device
// array instead of a caller-provided workspace.  Every GPU the library runs on holds its own copy of
// the array at its own address until the process ends; the address is looked up once per device, with
// that device current, and from then on only that pointer is used on the host side (kernel arguments):
// the array's name itself is no device address in host code.
static __device__ __align__(256) unsigned char scratch[GRACE_STATIC_SCRATCH_BYTES];

static int static_scratch(void **out) {
    constexpr int MAX_DEVICES = 64;
    static std::mutex mu;
    static void *ptr[MAX_DEVICES] = {nullptr};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(GRACE_EHIP, "route_permute_static: hipGetDevice: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= MAX_DEVICES) return fail(GRACE_EHIP, "route_permute_static: device %d not supported", dev);
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return fail(GRACE_EHIP, "route_permute_static: hipGetSymbolAddress: %s", hipGetErrorString(e));
        ptr[dev] = p;
    }
    *out = ptr[dev];
    return GRACE_OK;
}

extern "C" int grace_route_permute_static(const grace_table *table, int32_t local_rank, grace_policy policy,
                                          const float *logits, int32_t T, int32_t E, int32_t k, int32_t renorm,
                                          const uint32_t *rr_in, uint32_t *rr_out, int32_t *topk_expert, float *topk_weight,
                                          int32_t *topk_inst, int32_t *expert_count, const void *x, int32_t d,
                                          grace_dtype dt, int32_t *perm_pos, int32_t *perm_src, int32_t *inst_off,
                                          int32_t *rank_off, int32_t *node_off, void *xp, void *stream) {
    if (!table) return fail(GRACE_EINVAL, "route_permute_static: table is null");
    void *ws = nullptr;
    int rc = static_scratch(&ws);
    if (rc != GRACE_OK) return rc;
    rc = check_route_args(table, local_rank, policy, logits, T, E, k, rr_in, rr_out, topk_expert, topk_weight, topk_inst,
                          expert_count, ws);
    if (rc != GRACE_OK) return rc;
    rc = check_permute_args(table, topk_inst, T, k, x, d, dt, perm_pos, perm_src, inst_off, rank_off, node_off, xp, ws);
    if (rc != GRACE_OK) return rc;
    const size_t need = route_permute_ws_bytes(T, E, k, table->I);
    if (need > (size_t)GRACE_STATIC_SCRATCH_BYTES)
        return fail(GRACE_ESHAPE,
                    "route_permute_static: T=%d, E=%d, k=%d, I=%d need %zu bytes of scratch, the static buffer holds %zu; "
                    "use grace_route_permute with a workspace",
                    T, E, k, table->I, need, (size_t)GRACE_STATIC_SCRATCH_BYTES);
    // nothing in the scratch has to start at zero: every kernel of the call writes the histogram
    // rows and counters it later reads (the top-k kernel clears the permutation's counters)
    return route_permute_impl(table, local_rank, policy, logits, T, E, k, renorm, rr_in, rr_out, topk_expert, topk_weight,
                              topk_inst, expert_count, x, d, dt, perm_pos, perm_src, inst_off, rank_off, node_off, xp, ws,
                              stream);
}
