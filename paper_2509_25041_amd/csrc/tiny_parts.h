// Weights of all segments of a few rows by one workgroup, for some columns: the segments' parts of K ("items") are dealt to the
// wavefronts in turn, and each walks its items with DEPTH steps of 128 bytes of K in flight across their ends.
#pragma once
#include <algorithm>

#include "gemm_common.h"

namespace grace {

constexpr int PART_WAVES = 8, PART_THREADS = 64 * PART_WAVES;

// Parts of K per segment (their logarithm): enough items for the wavefronts, of two steps or more.
__device__ __forceinline__ int parts_log_of(int segments, int steps) {
    int p = segments <= 4 ? 3 : segments <= 16 ? 2 : segments <= 32 ? 1 : 0;
    while (p > 0 && steps < 2 << p) --p;
    return p;
}
inline int parts_most(int S, int n_shared) { return std::max(64, S + n_shared); }   // items: parts_log_of leaves 64 or one per segment

// A fragment of 16 weight rows holds 8, those of the upper half the second 64 bytes of their step: whole lines are loaded.  OCTETS, up to 8 activation
// rows: the activations' fragment holds them likewise, and the products of unlike halves are not looked at.  Else two fragments hold 16
// rows, a half of the step each, and half of their sums are not looked at.  Activations come from L2, but their loads take places of the
// weights' (16 tokens, d = 2048, f = 768, 5 segments, gate+up with two fragments 17.2 us, in octets, a second where needed, 16.6, without any 13.9).
// (Workgroups that begin an item at different steps, as the 96-row kernel's do, are no faster here: 0.98 to 1.02, 140 layer steps.)
//
// begin(segment): what load works on from here on; load(byte of K, NB weight fragments, activation fragments); leave(item, weight
// fragment, sum): weight rows 4 q to 4 q + 3 in lanes with q = lane / 16 < 2, activation row lane % 16 (OCTETS: below 8).
template <int EL, int NB, int DEPTH, bool OCTETS, typename Begin, typename Load, typename Leave>
__device__ __forceinline__ void walk_parts(int wave, int items, int parts_log, int steps, Begin begin, Load load_step, Leave leave) {
    const int parts = 1 << parts_log;
    auto start = [&](int item) { return ((item & (parts - 1)) * steps) >> parts_log; };
    auto end = [&](int item) { return (((item & (parts - 1)) + 1) * steps) >> parts_log; };
    constexpr int NA = OCTETS ? 1 : 2;   // activation fragments
    u32x4_t rb[DEPTH][NB], ra[DEPTH][NA];
    int next = wave, step = 0, last = 0;   // what is loaded next
    auto open = [&]() {
        if (next >= items) return;
        step = start(next);
        last = end(next);
        begin(next >> parts_log);
    };
    auto load = [&](int p) {
        if (next >= items) return;   // uniform
        load_step(step << 7, rb[p], ra[p]);
        __builtin_amdgcn_sched_barrier(0);
        if (++step == last) {
            next += PART_WAVES;
            open();
        }
    };
    f32x4_t acc[NB][NA];
    auto clear = [&]() {
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int h = 0; h < NA; ++h) acc[b][h] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    };
    auto mma = [&](int p, int h) {
        if constexpr (EL == 2) {
#pragma unroll
            for (int b = 0; b < NB; ++b)
                acc[b][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, rb[p][b]), __builtin_bit_cast(bf16x8_t, ra[p][h]), acc[b][h], 0, 0, 0);
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v)   // outermost: neighbours do not wait for each other's sums
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    acc[b][h] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(rb[p][b][v]), __uint_as_float(ra[p][h][v]), acc[b][h], 0, 0, 0);
        }
    };
    open();
    int item = wave, left = 0;   // in hand
    auto turn_to_item = [&]() {
        if (item >= items) return;
        left = end(item) - start(item);
    };
    turn_to_item();
    clear();
#pragma unroll
    for (int p = 0; p < DEPTH; ++p) load(p);
    while (item < items) {
#pragma unroll
        for (int p = 0; p < DEPTH; ++p) {
            if (item >= items) break;
            mma(p, 0);
            if constexpr (!OCTETS) mma(p, 1);
            load(p);
            if (--left == 0) {
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    f32x4_t sum;   // both halves' sums
#pragma unroll
                    for (int v = 0; v < 4; ++v) sum[v] = acc[b][0][v] + __shfl_xor(acc[b][NA - 1][v], OCTETS ? 40 : 32, 64);
                    leave(item, b, sum);
                }
                clear();
                item += PART_WAVES;
                turn_to_item();
            }
        }
    }
}

}  // namespace grace
