// The experts' gate+up projection and the dispatch of the smallest batches as one launch (ffn_tiny.hip).
#pragma once
#include "gemm_common.h"
#include "route_tiny.h"

namespace grace {

struct TinyUp {
    TinyArgs dispatch;
    GemmArgs up;              // A: the tokens; out: the hidden activation, T rows for each slot
    const uint4 *slot_span;   // of each local slot: its expert; its interval of polling weights among all instances of the expert, and their sum
    int slot0;                // instance id of the first one
    int several;              // the replica pick is among all instances (else every local expert's requests are the local instance's)
    int n_strips;
    GemmArgs shared;          // shared experts' gate+up projection by the same launch (shared_strips 0: none)
    int shared_strips;
    int piece_rows;           // fp32, more than 64 tokens: workgroups per that many rows at most (the launcher's)
};

// The record that the down projection's launch reads (share_record).
__device__ __forceinline__ void tiny_share_record(const TinyUp &a, const TinyLds &s) {
    if (!a.up.share_state || blockIdx.x != 0 || threadIdx.x != 0) return;
    int32_t *const state = a.up.share_state;
    state[0] = state[4];
    state[1] = state[5];
    state[4] = s.ioff[a.slot0];
    state[5] = s.ioff[a.slot0 + a.up.S];
}

// Tokens (bits of `mask`, cleared before, with a barrier behind) that chose expert e.  VPL: experts per lane; up to 32 experts a wavefront
// looks at several tokens at a time.
template <int VPL>
__device__ __forceinline__ void tokens_of(const TinyArgs &d, int e, uint32_t *mask) {
    constexpr int AHEAD = VPL > 2 ? 4 : VPL > 1 ? 8 : 16;   // tokens (or groups of them) whose logits are in flight
    const int lane = (int)threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), waves = (int)blockDim.x >> 6;
    const int shift = VPL > 1 || d.E > 32 ? 6 : max(1, bits_for(d.E)), per = 64 >> shift, width = 1 << shift;   // lanes per token
    const int col = lane & (width - 1), of = lane >> shift, count = (d.T + per - 1) / per;
    for (int i0 = wave; i0 < count; i0 += AHEAD * waves) {
        float raw[AHEAD][VPL];
#pragma unroll
        for (int i = 0; i < AHEAD; ++i)
#pragma unroll
            for (int v = 0; v < VPL; ++v) {
                const int t = (i0 + i * waves) * per + of;
                raw[i][v] = t < d.T && col + 64 * v < d.E ? d.logits[(size_t)t * d.E + col + 64 * v] : 0.0f;
            }
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) {
            const int t0 = (i0 + i * waves) * per;
            if (t0 >= d.T) break;   // uniform
            uint32_t key[VPL], own = 0;
#pragma unroll
            for (int v = 0; v < VPL; ++v) {
                key[v] = ordered_bits(raw[i][v] == 0.0f ? 0.0f : not_all_ones(raw[i][v]));
                if (v == e >> 6) own = key[v];
            }
            own = (uint32_t)__shfl((int)own, (of << shift) + (e & (width - 1)), 64);
            uint32_t bits;
            if (VPL > 1 || per == 1) {
                int ahead = 0;
#pragma unroll
                for (int v = 0; v < VPL; ++v) {
                    const int o = lane + 64 * v;
                    ahead += (int)__popcll(__ballot(o < d.E && (key[v] > own || (key[v] == own && o < e))));
                }
                bits = ahead < d.k ? 1u : 0u;
            } else {
                const uint64_t ahead = __ballot(col < d.E && (key[0] > own || (key[0] == own && col < e)));
                const uint64_t mine = (ahead >> ((lane << shift) & 63)) & ((1ull << width) - 1);   // (of token t0 + lane)
                bits = (uint32_t)__ballot(lane < per && t0 + lane < d.T && (int)__popcll(mine) < d.k);
            }
            if (lane == 0 && bits) atomicOr(&mask[t0 >> 5], bits << (t0 & 31));   // (per is at most 32 and divides t0)
        }
    }
}

struct TinyRows {
    uint32_t mask[TINY_MAX_T_TOP2 / 32];
    uint64_t kept[TINY_MAX_T_TOP2 / 64];
    int16_t list[TINY_MAX_T_TOP2];
};
constexpr int ROWS_BYTES = (sizeof(TinyRows) + 15) / 16 * 16;

// Tokens whose assignment to the expert of instance g0 + slot is that instance's, in order, in s.list; returns how many (uniform).
template <int VPL>
__device__ __forceinline__ int rows_of_slot(const TinyUp &a, int slot, TinyRows &s) {
    const TinyArgs &d = a.dispatch;
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const uint4 span = a.slot_span[slot];
    const int e = __builtin_amdgcn_readfirstlane((int)span.x);
    if (tid < TINY_MAX_T_TOP2 / 32) s.mask[tid] = 0u;
    if (tid < TINY_MAX_T_TOP2 / 64) s.kept[tid] = 0ull;
    __syncthreads();
    tokens_of<VPL>(d, e, s.mask);
    __syncthreads();
    bool mine = tid < d.T && (s.mask[tid >> 5] >> (tid & 31) & 1u);   // a thread per token
    if (a.several) {
        // request number -> instance: this one's if the number falls into its interval
        uint32_t number = (d.rr_in ? d.rr_in[e] : 0u) % span.w;
#pragma unroll
        for (int w = 0; w < TINY_MAX_T_TOP2 / 32; ++w) {
            const uint32_t before = w < tid >> 5 ? 0xFFFFFFFFu : w == tid >> 5 ? (1u << (tid & 31)) - 1u : 0u;
            number += (uint32_t)__popc(s.mask[w] & before);
        }
        number %= span.w;
        mine = mine && number >= span.y && number < span.z;
    }
    const uint64_t kept = __ballot(mine);
    if (lane == 0 && tid < TINY_MAX_T_TOP2) s.kept[tid >> 6] = kept;
    __syncthreads();
    int before = (int)__popcll(kept & lanemask_lt()), n = 0;
#pragma unroll
    for (int w = 0; w < TINY_MAX_T_TOP2 / 64; ++w) {
        const int c = (int)__popcll(s.kept[w]);
        n += c;
        before += w < tid >> 6 ? c : 0;
    }
    if (mine) s.list[before] = (int16_t)tid;
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(n);
}

// waves: per workgroup; pieces: more than 64 tokens (fp32).  The caller checks the launch, and allows the kernel LDS past 64 KB.
int tiny_up_lds(int T, int waves, bool pieces);   // bytes
const void *tiny_up_kernel_of(grace_dtype dt, int T, int E, bool pieces);
void launch_tiny_up(const TinyUp &a, grace_dtype dt, int waves, bool pieces, int n_cu, hipStream_t st);
// workgroups of the projection (the dispatch's T are extra), 0: too many tiles
int64_t tiny_up_mid_blocks(int S, int K, int n_strips, int n_cu);
// up to 96 tokens
void launch_tiny_up_mid(const TinyUp &a, int n_cu, hipStream_t st);

// K in whole 128-byte lines (ffn_tiny_cols.hip)
constexpr int TINY_COLS_T = 8;   // tokens
void launch_tiny_cols(const TinyUp &a, grace_dtype dt, int n_cu, hipStream_t st);

// The down projections and the combine of up to TINY_DOWN_T tokens (ffn_tiny_down.hip).
constexpr int TINY_DOWN_T = 16;
struct TinyDown {
    GemmArgs experts, shared;   // hidden activations laid out by slots; the shared experts' K axis is cut in segments of K
    const int32_t *perm_pos;
    const float *weight;
    void *out;
    int T, k, n_shared;
    int items_most;   // (the launcher's)
};
int tiny_down_lds(int T, int k, int S, int n_shared, int N, int n_cu);   // bytes
int tiny_down_blocks(int N, int n_cu);   // workgroups
const void *tiny_down_kernel_of(grace_dtype dt, int T, int N, int n_cu);
void launch_tiny_down(const TinyDown &a, grace_dtype dt, int lds, int n_cu, hipStream_t st);

}  // namespace grace
