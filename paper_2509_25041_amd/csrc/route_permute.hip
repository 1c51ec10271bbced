// grace_route_permute: grace_route followed by grace_permute as one call.
//
//   1. topk_kernel / topk_lanes_kernel (route.hip): choices, gate weights, a histogram of the chosen experts per chunk of tokens
//   2. place_kernel: request counters, replica pick (Algorithm 4 tier + weighted round-robin), offsets per instance / rank / node
//      and the stable position of every assignment in (node, rank, slot) order (Section 5)
//   3. scatter_rows_kernel (permute.hip): the rows
// The smallest batches take a single launch (route_permute_tiny_kernel).
// Outputs are identical either way (all integer work is exact and order-independent).
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "bf16.h"
#include "common.h"
#include "route_device.h"
#include "route_tiny.h"
#include "stable_sort.h"
#include "wave_utils.h"

namespace grace {

// Index work behind the top-k gate, one launch.  A request's number c among its expert's requests decides its instance (c mod W falls into
// a candidate's interval of cumulative polling weights) and, as every instance belongs to one expert, also how many earlier rows
// that instance has: of the requests 0 .. c - 1 those in the candidate's interval, (c / W) w + clamp(c mod W - first, 0, w).  So neither rows per
// instance nor a second ranking by instance are needed: the gate's histograms of experts give every workgroup the totals (the
// offsets) and the requests before its own tokens, and one ranking by expert gives instances and positions alike.  Bound by latency: the
// sums of the histogram rows, then four barriers.  A kernel for the picks and one for the positions -> this one, us: 1000 tokens of 64
// experts, k = 8 15.2 -> 9.2, 3001, k = 6 13.6 -> 7.9, 7001 of 128, k = 8 19.6 -> 10.7, 32768 of 64, k = 6 28.1 -> 12.3; a single workgroup for both
// -> this one: 512 tokens, k = 8 11.0 -> 6.4, 1000, k = 2 8.7 -> 7.3.
//
// A workgroup takes rows_per_block rows of the histogram, in rounds of PLACE_THREADS assignments.
constexpr int PLACE_THREADS = 512, PLACE_WAVES = PLACE_THREADS / 64;
constexpr int PLACE_LDS_CANDS = 1024;     // candidates of one view that are kept in LDS (else read from memory)

// Of requests number 0 .. c - 1 of an expert with weight sum W, those that the candidate with the interval [first, first + w) gets.
__device__ __forceinline__ uint32_t requests_to(uint32_t turns, uint32_t rest, uint32_t first, uint32_t w) {
    return turns * w + (rest <= first ? 0u : min(rest - first, w));   // c = turns * W + rest
}

__global__ __launch_bounds__(PLACE_THREADS) void place_kernel(
    const int32_t *__restrict__ topk_expert, int64_t n_assign, int E, int k, const int32_t *__restrict__ hist, int nrows, int chunk_tokens,
    int rows_per_block, const int32_t *__restrict__ super_tot, const uint32_t *__restrict__ rr_in, uint32_t *__restrict__ rr_out,
    int32_t *__restrict__ expert_count, const int32_t *__restrict__ cand_ptr, const int32_t *__restrict__ cand_g,
    const uint32_t *__restrict__ cand_cum, int c_first, int n_cand, int I, int R, int N, const int32_t *__restrict__ rank_ptr,
    const int32_t *__restrict__ node_first_inst, int32_t *__restrict__ topk_inst, int32_t *__restrict__ perm_pos,
    int32_t *__restrict__ perm_src, int32_t *__restrict__ inst_off, int32_t *__restrict__ rank_off, int32_t *__restrict__ node_off) {
    __shared__ int32_t all[GRACE_MAX_EXPERTS], cnt[GRACE_MAX_EXPERTS];   // requests of each expert: in all, before the current round
    __shared__ uint32_t carried[GRACE_MAX_EXPERTS], start[GRACE_MAX_EXPERTS];   // number of its first one, as carried over; mod W
    __shared__ int32_t wcnt[PLACE_WAVES][GRACE_MAX_EXPERTS];             // match set sizes of a wavefront, then requests before it
    __shared__ int32_t s_ptr[GRACE_MAX_EXPERTS + 1], s_g[PLACE_LDS_CANDS];
    __shared__ uint32_t s_cum[PLACE_LDS_CANDS];
    __shared__ int32_t off[GRACE_MAX_INSTANCES + 1], wave_sum[PLACE_WAVES];
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6, blk = (int)blockIdx.x;
    const int row0 = blk * rows_per_block;
    const int64_t per_block = (int64_t)rows_per_block * chunk_tokens * k, a0 = blk * per_block, a1 = min(n_assign, a0 + per_block);
    // the first round's experts and the candidates are in flight while the histogram rows are summed
    const int e_first = a0 + tid < a1 ? topk_expert[a0 + tid] : -1;
    const bool in_lds = n_cand <= PLACE_LDS_CANDS;   // uniform
    constexpr int CANDS = PLACE_LDS_CANDS / PLACE_THREADS;
    static_assert(GRACE_MAX_EXPERTS + 1 <= PLACE_THREADS && PLACE_LDS_CANDS % PLACE_THREADS == 0, "one offset, whole entries per thread");
    const int32_t st_ptr = tid <= E ? cand_ptr[tid] : 0;
    const uint32_t rr_own = rr_in && tid < E ? rr_in[tid] : 0u;
    int32_t st_g[CANDS];
    uint32_t st_cum[CANDS];
#pragma unroll
    for (int q = 0; q < CANDS; ++q) {
        const int i = tid + q * PLACE_THREADS;
        st_g[q] = in_lds && i < n_cand ? cand_g[c_first + i] : 0;
        st_cum[q] = in_lds && i < n_cand ? cand_cum[c_first + i] : 0u;
    }
    for (int i = tid; i < E; i += PLACE_THREADS) all[i] = cnt[i] = 0;
    for (int i = tid; i <= I; i += PLACE_THREADS) off[i] = 0;
    __syncthreads();
    if (super_tot) {   // sums of FOLD_SUPER rows each, then the rows behind the last whole one
        const int s = row0 / FOLD_SUPER;
        block_add_rows<PLACE_THREADS>(super_tot, 0, (nrows + FOLD_SUPER - 1) / FOLD_SUPER, E, all, tid, cnt, s);
        block_add_rows<PLACE_THREADS>(hist, s * FOLD_SUPER, row0, E, cnt, tid);
    } else {
        block_add_rows<PLACE_THREADS>(hist, 0, nrows, E, all, tid, cnt, row0);
    }
    if (tid <= E) s_ptr[tid] = in_lds ? st_ptr - c_first : st_ptr;
    if (tid < E) carried[tid] = rr_own;
#pragma unroll
    for (int q = 0; q < CANDS; ++q) {
        const int i = tid + q * PLACE_THREADS;
        if (in_lds && i < n_cand) {
            s_g[i] = st_g[q];
            s_cum[i] = st_cum[q];
        }
    }
    const int32_t *const t_g = in_lds ? s_g : cand_g;
    const uint32_t *const t_cum = in_lds ? s_cum : cand_cum;
    // sizes of the match sets of 64 assignments, in the wavefront's row of wcnt (its LDS operations execute in order)
    const int nbits = bits_for(E);
    bool valid;
    int e;
    uint64_t same;
    auto match = [&](int e_raw) {
        valid = (unsigned)e_raw < (unsigned)E;   // -1 past the end
        e = valid ? e_raw : 0;
        for (int i = lane; i < E; i += 64) wcnt[wave][i] = 0;
        same = wave_match((uint32_t)e, valid, nbits);
        if (valid && is_last_of(same)) wcnt[wave][e] = (int32_t)__popcll(same);
    };
    auto scan_waves = [&]() {
        for (int i = tid; i < E; i += PLACE_THREADS) {
            int32_t run = cnt[i];
#pragma unroll
            for (int w = 0; w < PLACE_WAVES; ++w) {
                const int32_t c = wcnt[w][i];
                wcnt[w][i] = run;
                run += c;
            }
            cnt[i] = run;
        }
    };
    match(e_first);
    __syncthreads();
    // ---- rows of every instance: several threads per expert, a candidate each
    const int subs = PLACE_THREADS / E, e_own = tid / subs;
    if (e_own < E) {
        const int cb = s_ptr[e_own], ce = s_ptr[e_own + 1];
        const uint32_t W = t_cum[ce - 1];
        const uint32_t first_number = carried[e_own] % W;
        if (tid % subs == 0) start[e_own] = first_number;
        const uint32_t end = first_number + (uint32_t)all[e_own];   // < 2^31 + 2^26
        const uint32_t turns = end / W, rest = end % W;
        for (int i = cb + tid % subs; i < ce; i += subs) {
            const uint32_t lo = i > cb ? t_cum[i - 1] : 0u, w = t_cum[i] - lo;
            off[t_g[i]] = (int32_t)(requests_to(turns, rest, lo, w) - requests_to(0u, first_number, lo, w));
        }
        if (blk == 0 && tid % subs == 0) {
            expert_count[e_own] = all[e_own];
            if (rr_out) rr_out[e_own] = rest;
        }
    }
    scan_waves();
    __syncthreads();
    // ---- offsets: exclusive scan over the instances
    int32_t *first = off;   // first row of every instance
    if (I <= MAX_KEYS) {
        // four per lane, by every wavefront for itself: two barriers fewer (128 tokens, k = 8, the whole call 12.15 -> 11.8 us)
        constexpr int STRIDE = MAX_KEYS + 4;
        static_assert((PLACE_WAVES + 1) * STRIDE <= GRACE_MAX_INSTANCES, "a copy per wavefront behind the totals");
        first = off + (wave + 1) * STRIDE;
        int32_t c[4], sum = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            c[q] = lane * 4 + q < I ? off[lane * 4 + q] : 0;
            sum += c[q];
        }
        const int32_t incl = wave_scan_add(sum);
        int32_t run = incl - sum;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            first[lane * 4 + q] = run;
            run += c[q];
        }
        if (lane == 63) first[MAX_KEYS] = run;
        wave_ctr_fence();   // the wavefront's LDS operations execute in order
    } else {
        // consecutive ones per thread
        const int per = (I + PLACE_THREADS - 1) / PLACE_THREADS, i0 = min(I, tid * per), i1 = min(I, i0 + per);
        int32_t sum = 0;
        for (int i = i0; i < i1; ++i) sum += off[i];
        const int32_t incl = wave_scan_add(sum);
        if (lane == 63) wave_sum[wave] = incl;
        __syncthreads();
        int32_t run = incl - sum;
#pragma unroll
        for (int w = 0; w < PLACE_WAVES; ++w) run += w < wave ? wave_sum[w] : 0;
        for (int i = i0; i < i1; ++i) {
            const int32_t c = off[i];
            off[i] = run;
            run += c;
        }
        if (tid == PLACE_THREADS - 1) off[I] = run;
        __syncthreads();
    }
    if (blk == 0) {
        for (int i = tid; i <= I; i += PLACE_THREADS) inst_off[i] = first[i];
        for (int r = tid; r <= R; r += PLACE_THREADS) rank_off[r] = first[rank_ptr[r]];
        for (int n = tid; n <= N; n += PLACE_THREADS) node_off[n] = first[node_first_inst[n]];
    }
    // ---- instances and positions
    const uint64_t lt = lanemask_lt();
    for (int64_t b0 = a0;;) {
        const int64_t a = b0 + tid;
        if (valid) {
            const int cb = s_ptr[e], ce = s_ptr[e + 1];
            const uint32_t from = start[e], W = t_cum[ce - 1], c = from + (uint32_t)wcnt[wave][e] + (uint32_t)__popcll(same & lt);
            const uint32_t turns = c / W, rest = c - turns * W;
            uint32_t lo = 0, hi = t_cum[cb];
            int s = cb;
            while (s < ce - 1 && hi <= rest) {
                lo = hi;
                hi = t_cum[++s];
            }
            const int g = t_g[s];
            const int64_t pos = (int64_t)first[g] + (int32_t)(requests_to(turns, rest, lo, hi - lo) - requests_to(0u, from, lo, hi - lo));
            topk_inst[a] = g;
            const bool inside = pos >= 0 && pos < n_assign;   // (always, unless the gate left an entry unwritten: logits that are all NaN)
            perm_pos[a] = inside ? (int32_t)pos : -1;
            if (inside) perm_src[pos] = (int32_t)a;
        } else if (a < a1) {
            perm_pos[a] = -1;   // expert id outside the table: no row
        }
        b0 += PLACE_THREADS;
        if (b0 >= a1) break;
        __syncthreads();   // wcnt has been read
        match(b0 + tid < a1 ? topk_expert[b0 + tid] : -1);
        __syncthreads();
        scan_waves();
        __syncthreads();
    }
}

// The smallest batches: top-k, index work and row movement in one launch (route_tiny.h).  Three launches of 2 to 7 us each wait for one
// another's first loads there, while all the index work of 64 tokens is a few microseconds for one workgroup.  A wavefront takes a token in
// the gate, four past 16 tokens, or 64 of up to 16 experts where four would take more than one pass (256 tokens of 8 experts, k = 2, four at a time 9.5, 64 at a time 6.2 us).
// Layer steps, the three launches -> this one (1, 16, 64 tokens): 64 experts, k = 8 24.3 -> 20.8, 30.6 -> 25.0, 38.0 -> 33.9 us; 8 experts, k = 2
// 22.8 -> 17.8, 30.8 -> 27.2, 34.9 -> 30.5 us; 128 experts, k = 8 22.8 -> 18.8, 31.1 -> 24.0 us.  Where the line lies: every workgroup
// repeats the gate of all tokens, so the call (replayed from a graph) gains less with each.  96 tokens, 64 experts, k = 3, 4, 5, 6, 8: three
// launches as the next larger batch takes them 10.4, 10.4, 11.0, 11.2, 11.8, this one 7.5, 8.2, 8.6, 9.4, 10.5 us; 85 tokens, k = 12 is the most
// assignments.  Past 96 tokens k = 6 and 8 are about even in a step (128 tokens 56.7 -> 57.6, 39.1 -> 38.3 us).  256 tokens with k = 1, 2, where four
// passes of the wavefronts of four tokens end: 9.1, 10.0 to 10.6 against 10.9, 10.4 to 11.0 us.  128 and 256 experts, 32 tokens, k = 8, two passes: 9.5 and 11.4
// against 12.3 and 14.0 us (33 tokens); four tokens by rows there 33 tokens 32.1 -> 32.2, 64 tokens 34.9 -> 36.1 us a step.
template <int VPL, Gate GATE, int PASSES>
__global__ __launch_bounds__(64 * TINY_MAX_WAVES) void route_permute_tiny_kernel(const TinyArgs d) {
    __shared__ TinyLds lds;
    tiny_dispatch<VPL, GATE, PASSES, true>(d, (int)blockIdx.x, lds);
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
    const int view = policy == GRACE_POLICY_WRR ? table->R : local_rank;
    const int32_t *cand_ptr = table->d_cand_ptr + (size_t)view * E;
    if (tiny_batch(T, k, E, table->I)) {
        int waves = 4;   // a thread per expert and instance, a wavefront per 64 assignments and, up to the most, per token or four
        const bool lanes = E <= TINY_LANE_E && T > 4 * TINY_MAX_WAVES, rows = E <= 64 && T > TINY_MAX_WAVES && !lanes;
        while (!lanes && waves < TINY_MAX_WAVES && waves * (rows ? 4 : 1) < T) waves *= 2;
        while (waves * 64 < T * k) waves *= 2;
        auto launch = [&](auto vpl) {
            constexpr int VPL = decltype(vpl)::value;
            auto *kern = route_permute_tiny_kernel<VPL, Gate::WAVE, 1>;
            if constexpr (VPL == 1) {
                if (lanes) kern = route_permute_tiny_kernel<1, Gate::LANES, 1>;
                else if (rows) kern = T <= 4 * waves ? route_permute_tiny_kernel<1, Gate::ROWS, 1> : T <= 8 * waves ? route_permute_tiny_kernel<1, Gate::ROWS, 2>
                                                                                                                 : route_permute_tiny_kernel<1, Gate::ROWS, 4>;
            } else if (T > waves) {
                kern = route_permute_tiny_kernel<VPL, Gate::WAVE, 2>;
            }
            kern<<<T, waves * 64, 0, st>>>(tiny_args(table, local_rank, policy, logits, T, k, renorm, rr_in, rr_out, topk_expert, topk_weight,
                                                     topk_inst, expert_count, x, d, dt, perm_pos, perm_src, inst_off, rank_off, node_off, xp));
        };
        if (E <= 64) launch(std::integral_constant<int, 1>{});
        else if (E <= 128) launch(std::integral_constant<int, 2>{});
        else if (E <= 192) launch(std::integral_constant<int, 3>{});
        else launch(std::integral_constant<int, 4>{});
        GRACE_LAUNCH_CHECK("route_permute_tiny_kernel");
        return GRACE_OK;
    }
    const int chunk_tokens = route_chunk_tokens(T), nrows = (int)ceil_div(T, chunk_tokens), mode = fold_mode(table, nrows, E);
    if (mode == 0) {   // no tokens, or so many that the histograms are scanned by launches of their own
        rc = grace_route(table, local_rank, policy, logits, T, E, k, renorm, rr_in, rr_out, topk_expert, topk_weight,
                         topk_inst, expert_count, ws, stream);
        if (rc != GRACE_OK) return rc;
        return grace_permute(table, topk_inst, T, k, x, d, dt, perm_pos, perm_src, inst_off, rank_off, node_off, xp, ws,
                             stream);
    }
    int32_t *hist = (int32_t *)ws;
    rc = launch_topk(logits, T, E, k, renorm, topk_expert, topk_weight, hist, st);
    if (rc != GRACE_OK) return rc;
    const int32_t *super_tot = nullptr;
    if (mode == 2) {
        int32_t *sums = (int32_t *)((char *)ws + align_up((size_t)nrows * E * 4, 256));
        super_sum_kernel<<<(unsigned)ceil_div(nrows, FOLD_SUPER), SUPER_THREADS, 0, st>>>(hist, nrows, E, sums);
        GRACE_LAUNCH_CHECK("super_sum_kernel");
        super_tot = sums;
    }
    const int rows_per_block = std::max(1, PLACE_THREADS / (k * chunk_tokens));
    place_kernel<<<(unsigned)ceil_div(nrows, rows_per_block), PLACE_THREADS, 0, st>>>(
        topk_expert, (int64_t)T * k, E, k, hist, nrows, chunk_tokens, rows_per_block, super_tot, rr_in, rr_out, expert_count, cand_ptr,
        table->d_cand_g, table->d_cand_cum, table->cand_view[view], table->cand_view[view + 1] - table->cand_view[view], table->I, table->R,
        table->N, table->d_rank_ptr, table->d_node_first_inst, topk_inst, perm_pos, perm_src, inst_off, rank_off, node_off);
    GRACE_LAUNCH_CHECK("place_kernel");
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
    // nothing in the scratch has to start at zero: the call's kernels write every histogram row and sum that a later one reads
    return route_permute_impl(table, local_rank, policy, logits, T, E, k, renorm, rr_in, rr_out, topk_expert, topk_weight,
                              topk_inst, expert_count, x, d, dt, perm_pos, perm_src, inst_off, rank_off, node_off, xp, ws,
                              stream);
}
