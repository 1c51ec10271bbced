// grace_send_lists: de-duplicated hierarchical send lists and traffic counters.
//
// The two-stage dispatch of Section 5 forwards a token once per destination even
// when several of its experts live there.  For the tokens of
// local_rank this builds, per destination rank and per destination node, the
// ascending list of distinct tokens that have at least one assignment there, the
// map that lets the receiver expand the unique rows back to one row per
// assignment, and the token counts the paper's traffic metrics are made of.
//
//   1. dedup_keys_kernel  one lane per assignment: its destination rank / node; the
//                         token's first assignment per destination keeps the
//                         destination as its sort key, the others get -1
//   2. stable counting sorts by rank key and by node key (stable_sort.h), one launch for both where each is one
//   3. expand_traffic_kernel  expansion map + traffic sums
// At most PERM_CHUNK assignments: send_lists_small_kernel does all of it in one workgroup.
//
// The lists are used by planning code that makes several short calls per batch, so launches count: with grace_route ahead and
// grace_permute behind, 16384 tokens of k = 4 take 74.4 -> 61.9 us with
// seven launches instead of ten (one for both sorts, no fills of the lists ahead of them), 9001 of k = 6 68.9 -> 57.7 us.
#include "common.h"
#include "stable_sort.h"

namespace grace {

// Keys of assignment a: its destination rank and node if it is its token's first choice there, else -1; counted.
__device__ __forceinline__ void dedup_keys(const int32_t *__restrict__ topk_inst, int64_t a, int k, int I,
                                           const int32_t *__restrict__ inst_rank, const int32_t *__restrict__ rank_node,
                                           int32_t *__restrict__ rank_key, int32_t *__restrict__ node_key,
                                           int32_t *__restrict__ first_idx, int32_t *rank_cnt, int32_t *node_cnt) {
    const int64_t t = a / k;
    const int j = (int)(a - t * k);
    const int32_t *row = topk_inst + t * k;
    const int g = row[j];
    if ((unsigned)g >= (unsigned)I) {  // id outside the table: no destination
        rank_key[a] = -1; node_key[a] = -1; first_idx[a] = -1;
        return;
    }
    const int r = inst_rank[g], nd = rank_node[r];
    int first_r = j;
    bool first_n = true;
    for (int jj = 0; jj < j; ++jj) {
        const int g2 = row[jj];
        if ((unsigned)g2 >= (unsigned)I) continue;
        const int r2 = inst_rank[g2];
        if (r2 == r && first_r == j) first_r = jj;
        if (rank_node[r2] == nd) first_n = false;
    }
    rank_key[a] = (first_r == j) ? r : -1;
    node_key[a] = first_n ? nd : -1;
    if (first_r == j) atomicAdd(&rank_cnt[r], 1);
    if (first_n) atomicAdd(&node_cnt[nd], 1);
    first_idx[a] = (int32_t)(t * k + first_r);
}

// One lane per assignment, one block per chunk of the sorts that follow: the block counts its own keys, which
// saves the sorts' histogram launches (4.2 us each at 65536 assignments).  node_hist may be null (not wanted).  The
// first blocks also clear the counters that expand_traffic_kernel accumulates into later in the same call (rows
// per destination rank, finished-block count).
__global__ __launch_bounds__(PERM_CHUNK) void dedup_keys_kernel(const int32_t *__restrict__ topk_inst, int64_t n_assign, int k,
                                                         int I, const int32_t *__restrict__ inst_rank,
                                                         const int32_t *__restrict__ rank_node,
                                                         int32_t *__restrict__ rank_key, int32_t *__restrict__ node_key,
                                                         int32_t *__restrict__ first_idx, int32_t *__restrict__ counters,
                                                         int n_counters, int R, int N, int32_t *__restrict__ rank_hist,
                                                         int32_t *__restrict__ node_hist) {
    __shared__ int32_t hist[2 * GRACE_MAX_RANKS];   // ranks, nodes
    for (int i = (int)threadIdx.x; i < R + N; i += PERM_CHUNK) hist[i] = 0;
    __syncthreads();
    const int64_t a = (int64_t)blockIdx.x * PERM_CHUNK + threadIdx.x;
    if (a < n_counters) counters[a] = 0;
    if (a < n_assign) dedup_keys(topk_inst, a, k, I, inst_rank, rank_node, rank_key, node_key, first_idx, hist, hist + R);
    __syncthreads();
    if ((int64_t)blockIdx.x * PERM_CHUNK >= n_assign) return;
    for (int i = (int)threadIdx.x; i < R; i += PERM_CHUNK) rank_hist[(size_t)blockIdx.x * R + i] = hist[i];
    if (!node_hist) return;
    for (int i = (int)threadIdx.x; i < N; i += PERM_CHUNK) node_hist[(size_t)blockIdx.x * N + i] = hist[R + i];
}

// traffic[] (below) from the list lengths and the rows of every destination rank, by a whole workgroup; acc: LDS.
template <typename ROWS>
__device__ __forceinline__ void traffic_sums(int R, int N, int local_rank, const int32_t *__restrict__ rank_node,
                                             const int32_t *rank_send_ptr, const int32_t *node_send_ptr, ROWS rows_of,
                                             unsigned long long *acc, int64_t *__restrict__ traffic) {
    if (threadIdx.x < 4) acc[threadIdx.x] = 0ull;
    __syncthreads();
    const int my_node = rank_node[local_rank];
    int my_first = 0;  // first rank of the own node (ranks are node-major)
    while (my_first < R && rank_node[my_first] != my_node) ++my_first;
    const int local_idx = local_rank - my_first;
    for (int r = (int)threadIdx.x; r < R; r += (int)blockDim.x) {
        const int nd = rank_node[r];
        const unsigned long long uniq = (unsigned long long)(rank_send_ptr[r + 1] - rank_send_ptr[r]);
        const unsigned long long rows = (unsigned long long)rows_of(r);
        if (nd != my_node) {
            atomicAdd(&acc[1], rows);
            // the peer of local_rank in node nd: same index inside the node (modulo the node's size)
            int first = r, size = 0;
            while (first > 0 && rank_node[first - 1] == nd) --first;
            while (first + size < R && rank_node[first + size] == nd) ++size;
            const int peer = first + local_idx % size;
            if (r != peer) atomicAdd(&acc[2], uniq);
        } else if (r != local_rank) {
            atomicAdd(&acc[2], uniq);
            atomicAdd(&acc[3], rows);
        }
    }
    for (int n = (int)threadIdx.x; n < N; n += (int)blockDim.x)
        if (n != my_node) atomicAdd(&acc[0], (unsigned long long)(node_send_ptr[n + 1] - node_send_ptr[n]));
    __syncthreads();
    if (threadIdx.x < 4) traffic[threadIdx.x] = (int64_t)acc[threadIdx.x];
}

// expand[a] = index of a's token in the send list of a's destination rank.
// traffic[0] cross-node tokens with de-duplication: sum over other nodes of their distinct tokens
// traffic[1] cross-node rows without (one per assignment)
// traffic[2] intra-node tokens with de-duplication: distinct tokens for the other ranks of the own
//            node plus, in every other node, for the ranks other than the peer that received stage 1
// traffic[3] intra-node rows of a flat dispatch: assignments to the other ranks of the own node
// rank_tail, node_tail (both or none): the lists, whose entries past their ends become -1.
// counters: [0, R) rows per destination rank (all blocks add their share: integer sums, exact in any
// order), [R] number of blocks that have added; the block that finishes last turns them into traffic[].
// EXPAND_CHUNK assignments per block: the blocks' sums meet on the same few addresses (65536 assignments, 8 ranks:
// 10.4 us with 256 per block).
constexpr int EXPAND_CHUNK = 1024;
__global__ __launch_bounds__(256) void expand_traffic_kernel(const int32_t *__restrict__ topk_inst, int64_t n_assign, int I,
                                                             int R, int N, int local_rank,
                                                             const int32_t *__restrict__ inst_rank,
                                                             const int32_t *__restrict__ rank_node,
                                                             const int32_t *__restrict__ first_idx,
                                                             const int32_t *__restrict__ send_pos,
                                                             const int32_t *__restrict__ rank_send_ptr,
                                                             const int32_t *__restrict__ node_send_ptr,
                                                             int32_t *__restrict__ expand, int64_t *__restrict__ traffic,
                                                             int32_t *__restrict__ counters, int32_t *__restrict__ rank_tail,
                                                             int32_t *__restrict__ node_tail) {
    __shared__ int32_t naive_rank[GRACE_MAX_RANKS];
    __shared__ unsigned long long acc[4];
    __shared__ int last_block;
    const int64_t a0 = (int64_t)blockIdx.x * EXPAND_CHUNK + threadIdx.x;
    if (traffic)
        for (int r = (int)threadIdx.x; r < R; r += 256) naive_rank[r] = 0;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < EXPAND_CHUNK / 256; ++q) {
        const int64_t a = a0 + q * 256;
        if (a >= n_assign) break;
        const int g = topk_inst[a];
        int32_t e = -1;
        if ((unsigned)g < (unsigned)I) {
            const int r = inst_rank[g];
            e = send_pos[first_idx[a]] - rank_send_ptr[r];
            if (traffic) atomicAdd(&naive_rank[r], 1);
        }
        expand[a] = e;
        if (rank_tail) {
            if (a >= rank_send_ptr[R]) rank_tail[a] = -1;
            if (a >= node_send_ptr[N]) node_tail[a] = -1;
        }
    }
    if (!traffic) return;
    __syncthreads();
    // The sums are performed (their old values have come back) before this block counts itself as finished; they
    // and the last block's reads are atomics at device scope, so no fence is needed, which would write back
    // and invalidate the L2 once per block (65536 assignments: 21.6 us with fences).
    for (int r = (int)threadIdx.x; r < R; r += 256) {
        const int32_t add = naive_rank[r];
        if (add) {
            const int32_t old = atomicAdd(&counters[r], add);
            asm volatile("" ::"v"(old) : "memory");
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) last_block = atomicAdd(&counters[R], 1) == (int)gridDim.x - 1;
    __syncthreads();
    if (!last_block) return;
    traffic_sums(R, N, local_rank, rank_node, rank_send_ptr, node_send_ptr,
                 [&](int r) { return atomicAdd(&counters[r], 0); },   // read at the L2, past this CU's cache
                 acc, traffic);
}

// At most one chunk of assignments, and as many ranks: a workgroup does everything in LDS, one launch instead of three
//
// (the same calls for 1 and 60 tokens of k = 8: 68 -> 49 us, half of it from the fills and the permutation's histogram).
constexpr int SMALL_LIST_RANKS = PERM_CHUNK;
__global__ __launch_bounds__(PERM_CHUNK) void send_lists_small_kernel(
    const int32_t *__restrict__ topk_inst, int n, int k, int I, int R, int N, int local_rank, const int32_t *__restrict__ inst_rank,
    const int32_t *__restrict__ rank_node, int32_t *__restrict__ rank_send_ptr, int32_t *__restrict__ rank_send_tok,
    int32_t *__restrict__ node_send_ptr, int32_t *__restrict__ node_send_tok, int32_t *__restrict__ expand,
    int64_t *__restrict__ traffic, int fill) {
    constexpr int WAVES = PERM_CHUNK / 64;
    __shared__ int32_t wcnt[WAVES][SMALL_LIST_RANKS];                        // keys of a wavefront, then those before it
    __shared__ int32_t roff[SMALL_LIST_RANKS + 1], noff[SMALL_LIST_RANKS + 1];   // list starts
    __shared__ int32_t dest_r[PERM_CHUNK], dest_n[PERM_CHUNK], where[PERM_CHUNK];
    __shared__ int32_t rows[SMALL_LIST_RANKS];
    __shared__ unsigned long long acc[4];
    const int a = (int)threadIdx.x, lane = a & 63, wave = a >> 6;
    const int g = a < n ? topk_inst[a] : -1;
    const bool to = (unsigned)g < (unsigned)I;
    const int r = to ? inst_rank[g] : -1, nd = to ? rank_node[r] : -1;
    dest_r[a] = r;
    dest_n[a] = nd;
    rows[a] = 0;
    __syncthreads();
    int first = a;
    bool first_n = true;
    for (int b = a - a % k; b < a; ++b) {
        if (dest_r[b] == r && first == a) first = b;
        if (dest_n[b] == nd) first_n = false;
    }
    if (to && traffic) atomicAdd(&rows[r], 1);
    auto sort = [&](int key, int nkeys, int32_t *off, int32_t *ptr, int32_t *tok) {   // position of this thread's key
        for (int i = lane; i < nkeys; i += 64) wcnt[wave][i] = 0;   // its own wavefront's row: in program order
        const bool valid = key >= 0;
        const uint64_t same = wave_match((uint32_t)max(key, 0), valid, bits_for(nkeys));
        if (valid && is_last_of(same)) wcnt[wave][key] = (int32_t)__popcll(same);
        __syncthreads();
        if (a < nkeys) {
            int32_t run = 0;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) {
                const int32_t c = wcnt[w][a];
                wcnt[w][a] = run;
                run += c;
            }
            off[a] = run;
        }
        __syncthreads();
        if (wave == 0) {
            int32_t carry = 0;
            for (int k0 = 0; k0 < nkeys; k0 += 64) {
                const int32_t c = k0 + lane < nkeys ? off[k0 + lane] : 0, incl = wave_scan_add(c);
                if (k0 + lane < nkeys) off[k0 + lane] = carry + incl - c;
                carry += __builtin_amdgcn_readlane(incl, 63);
            }
            if (lane == 0) off[nkeys] = carry;
        }
        __syncthreads();
        for (int i = a; i <= nkeys; i += PERM_CHUNK) ptr[i] = off[i];
        int32_t pos = -1;
        if (valid) {
            pos = off[key] + wcnt[wave][key] + (int32_t)__popcll(same & lanemask_lt());
            tok[pos] = a / k;
        }
        if (fill && a < n && a >= off[nkeys]) tok[a] = -1;
        return pos;
    };
    where[a] = sort(to && first == a ? r : -1, R, roff, rank_send_ptr, rank_send_tok);
    __syncthreads();   // before the next sort's counts, too
    if (a < n) expand[a] = to ? where[first] - roff[r] : -1;
    sort(to && first_n ? nd : -1, N, noff, node_send_ptr, node_send_tok);
    if (traffic) traffic_sums(R, N, local_rank, rank_node, roff, noff, [&](int r) { return rows[r]; }, acc, traffic);
}

static int bits(int nkeys) {
    int b = 0;
    while ((1 << b) < nkeys) ++b;
    return b;
}

static int sort_by_key(const grace_table *table, const int32_t *keys, int64_t n, int k, int nkeys, int32_t *hist, int32_t *base, int32_t *off,
                       int32_t *pos, int32_t *tok, hipStream_t st, bool hist_ready) {
    const char *failed = stable_sort_launch(table, keys, n, nkeys, k, hist, base, 0, 0, nullptr, nullptr, off, nullptr, nullptr,
                                            pos, tok, st, hist_ready);
    if (failed) return fail(GRACE_EHIP, "send_lists: launch of %s failed", failed);
    return GRACE_OK;
}

}  // namespace grace

using namespace grace;

static int send_lists(const grace_table *table, int32_t local_rank, const int32_t *topk_inst, int32_t T, int32_t k,
                      int32_t *rank_send_ptr, int32_t *rank_send_tok, int32_t *node_send_ptr, int32_t *node_send_tok, int32_t *expand,
                      int64_t *traffic, bool fill, void *ws, void *stream) {
    if (!table) return fail(GRACE_EINVAL, "send_lists: table is null");
    if (local_rank < 0 || local_rank >= table->R)
        return fail(GRACE_EINVAL, "send_lists: local_rank=%d outside [0,%d)", local_rank, table->R);
    if (T < 0 || k < 1) return fail(GRACE_EINVAL, "send_lists: T=%d, k=%d invalid", T, k);
    if ((int64_t)T * k > INT32_MAX) return fail(GRACE_ESHAPE, "send_lists: T*k exceeds 2^31-1");
    if (!rank_send_ptr || !node_send_ptr || !ws) return fail(GRACE_EINVAL, "send_lists: null offset or ws pointer");
    if (T > 0 && (!topk_inst || !rank_send_tok || !node_send_tok || !expand))
        return fail(GRACE_EINVAL, "send_lists: null device pointer");
    hipStream_t st = (hipStream_t)stream;
    const int64_t n = (int64_t)T * k;
    const int R = table->R, N = table->N, I = table->I;
    if (n > 0 && n <= PERM_CHUNK && std::max(R, N) <= SMALL_LIST_RANKS && fold_mode(table, 1, R) == 1) {
        send_lists_small_kernel<<<1, PERM_CHUNK, 0, st>>>(topk_inst, (int)n, k, I, R, N, local_rank, table->d_inst_rank, table->d_rank_node,
                                                          rank_send_ptr, rank_send_tok, node_send_ptr, node_send_tok, expand, traffic,
                                                          fill);
        GRACE_LAUNCH_CHECK("send_lists_small_kernel");
        return GRACE_OK;
    }
    const size_t seg = align_up((size_t)n * 4, 256);
    char *w = (char *)ws;
    int32_t *rank_key = (int32_t *)w, *node_key = (int32_t *)(w + seg), *first_idx = (int32_t *)(w + 2 * seg);
    int32_t *pos_r = (int32_t *)(w + 3 * seg), *pos_n = (int32_t *)(w + 4 * seg);
    const size_t nchunks = (size_t)ceil_div(n, PERM_CHUNK);
    int32_t *hist = (int32_t *)(w + 5 * seg);
    // both sorts' chunk histograms share the space of one over GRACE_MAX_RANKS keys; with nearly as many ranks and
    // nodes as that, the node sort counts its keys itself after the rank sort
    const size_t hist_bytes = align_up(nchunks * (size_t)GRACE_MAX_RANKS * 4, 256), rank_bytes = align_up(nchunks * (size_t)R * 4, 256);
    int32_t *node_hist = rank_bytes + nchunks * (size_t)N * 4 <= hist_bytes ? (int32_t *)((char *)hist + rank_bytes) : nullptr;
    int32_t *base = (int32_t *)(w + 5 * seg + align_up(nchunks * (size_t)GRACE_MAX_RANKS * 4, 256));
    // R per-rank row counters + 1 finished-block counter, behind the chunk histograms
    int32_t *counters = (int32_t *)(w + 5 * seg + 2 * align_up(nchunks * (size_t)GRACE_MAX_RANKS * 4, 256));
    {
        const int64_t lanes = std::max<int64_t>(n, R + 1);
        dedup_keys_kernel<<<(unsigned)ceil_div(lanes, PERM_CHUNK), PERM_CHUNK, 0, st>>>(
            topk_inst, n, k, I, table->d_inst_rank, table->d_rank_node, rank_key, node_key, first_idx, counters, R + 1, R, N, hist,
            node_hist);
        GRACE_LAUNCH_CHECK("dedup_keys_kernel");
    }
    if (node_hist && fold_mode(table, (int)nchunks, R) == 1 && fold_mode(table, (int)nchunks, N) == 1) {
        const KeySort ranks = {rank_key, R, bits(R), hist, nullptr, rank_send_ptr, pos_r, rank_send_tok};
        const KeySort nodes = {node_key, N, bits(N), node_hist, nullptr, node_send_ptr, pos_n, node_send_tok};
        key_pos_fold_pair_kernel<<<dim3((unsigned)nchunks, 2), POS_FOLD_THREADS, 0, st>>>(ranks, nodes, n, (int)nchunks, k);
        GRACE_LAUNCH_CHECK("key_pos_fold_pair_kernel");
    } else {
        int rc = sort_by_key(table, rank_key, n, k, R, hist, base, rank_send_ptr, pos_r, rank_send_tok, st, true);
        if (rc != GRACE_OK) return rc;
        rc = sort_by_key(table, node_key, n, k, N, node_hist ? node_hist : hist, base, node_send_ptr, pos_n, node_send_tok, st,
                         node_hist != nullptr);
        if (rc != GRACE_OK) return rc;
    }
    if (n > 0 || traffic) {
        expand_traffic_kernel<<<(unsigned)std::max<int64_t>(1, ceil_div(n, EXPAND_CHUNK)), 256, 0, st>>>(
            topk_inst, n, I, R, N, local_rank, table->d_inst_rank, table->d_rank_node, first_idx, pos_r, rank_send_ptr,
            node_send_ptr, expand, traffic, counters, fill ? rank_send_tok : nullptr, node_send_tok);
        GRACE_LAUNCH_CHECK("expand_traffic_kernel");
    }
    return GRACE_OK;
}

extern "C" int grace_send_lists(const grace_table *table, int32_t local_rank, const int32_t *topk_inst, int32_t T,
                                int32_t k, int32_t *rank_send_ptr, int32_t *rank_send_tok, int32_t *node_send_ptr,
                                int32_t *node_send_tok, int32_t *expand, int64_t *traffic, void *ws, void *stream) {
    return send_lists(table, local_rank, topk_inst, T, k, rank_send_ptr, rank_send_tok, node_send_ptr, node_send_tok, expand, traffic,
                      false, ws, stream);
}

extern "C" int grace_send_lists_fresh(const grace_table *table, int32_t local_rank, const int32_t *topk_inst, int32_t T,
                                      int32_t k, int32_t *rank_send_ptr, int32_t *rank_send_tok, int32_t *node_send_ptr,
                                      int32_t *node_send_tok, int32_t *expand, int64_t *traffic, void *ws, void *stream) {
    return send_lists(table, local_rank, topk_inst, T, k, rank_send_ptr, rank_send_tok, node_send_ptr, node_send_tok, expand, traffic,
                      true, ws, stream);
}
