// bf16 MFMA grouped GEMM for ordinary batches: 96 rows x 128 weight rows per workgroup, any K that is a multiple of 8.
//
// Between decode batches (gemm_stream.h) and prefill (gemm_bf16_persist.h) most row segments hold fewer rows than
// a tile of the large kernel, so the product is still bound by reading every weight once, while a few hot
// segments need the matrix cores.  256 x 256 tiles leave compute units without work there (16 segments of an
// expert width of 1024 make about 150 tiles) and one workgroup per compute unit waits alone for its weights.
//
// A workgroup of four wavefronts takes up to 96 rows of a segment and 128 weight rows (gate+up: 64 of each
// matrix); two fit a compute unit.  The wavefronts split the weight rows, and everything is loaded into registers
// AHEAD steps of 64 K ahead (weights in flight per compute unit: 128 KB, twice that for up to 32 rows), in whole
// 128-byte lines: 8 lanes per row.  Loading weights in the MFMA's own layout (row = lane % 16) instead touches a
// line per lane and makes the address unit the bound (decode batch of 512: 48 instead of 38 us for the gate+up
// projection).  One step ahead of its use a step's data goes to one of two LDS buffers: the activation rows,
// which all four wavefronts read, and each wavefront's own weights (16-byte chunk c of row r at
// c ^ ((r >> 1) & 7): no bank conflicts), with one barrier per step.  The order of fragment reads and MFMAs is
// fixed, so that a read has a pass of MFMAs to arrive.  Loads past K, past the piece's rows or past N are given
// an offset outside the buffer descriptor's range: they read nothing and give zeros, so every step is the same
// code whatever K is.
//
// Groups of four neighbouring strips walk K from different steps on, round and round: with all tiles at the same K, the
// rows' lines of that moment lie a row apart, and where a row is a multiple of 2 or 4 KB they fall on a few of the memory's
// channels (16 segments, d = 2048, f = 1024, cold weights, gate+up: 19 rows each 36.5 -> 28.1 us, 96 each 37.0 -> 29.5 us, 1024 rows with
// Zipf-shaped shares 43.5 -> 39.9 us; d = 4096, f = 3584, 8 segments of 19 rows 91.6 -> 82.0 us; rows of 2 KB and less are even).
// Single strips at different steps lose what they share of the activation rows in L2 (96 rows each 31 to 38 us).  A strip's
// step depends on its weights alone, so a row's result does not depend on the batch around it.
//
// Pieces of a segment have one size (a multiple of 16, at most 96).  Workgroups are numbered by segment, strip
// of weight rows, piece, and dealt to the XCDs in 64 runs of equal length (workgroups go to the XCDs round-robin):
// pieces that read the same weights run next to each other on one L2, and every XCD gets hot and cold segments
// (8 runs: 42 instead of 39 us on the batch of 512).
//
// Measured with cold weights, all segments in use (more than 1 GB of others between two uses; up / down projection, 256 x 256
// tiles and this kernel, us): 16 segments of d = 2048, f = 1024, 2236 rows with Zipf-shaped shares 50.1 / 26.2 and 41.7 /
// 25.9, 300 rows 41.6 / 24.5 and 32.3 / 19.5; f = 768, 985 rows 44.4 / 22.0 and 28.0 / 19.4; d = 4096, f = 14336, one
// segment of 64 rows 70.5 / 199.8 and 43.9 / 60.4, of 512 rows 99.5 / 193.8 and 188.5 / 125.1 (the choice takes large tiles
// for the first of the two).  Segments as a batch of 70 tokens has them, 11 of 16 in use 36.2 / 21.1 and 23.0 / 14.8, of 230
// tokens, 13 of 16 45.8 / 23.4 and 27.1 / 17.1.
// K that is no multiple of 64 took a kernel without prefetch before: 3001 rows, N = 2048, K = 2 x 352 58 -> 20 us.
#pragma once
#include <algorithm>
#include <type_traits>

#include "bf16.h"
#include "gemm_common.h"

namespace grace {
namespace mid {

constexpr int BM = 96, BK = 64, THREADS = 256;
constexpr int ROW_BYTES = BK * 2, A_BYTES = BM * ROW_BYTES, B_WAVE_BYTES = 32 * ROW_BYTES, LDS_BYTES = 2 * A_BYTES + 8 * B_WAVE_BYTES;

template <bool FUSED_UP>
struct Shape {
    static constexpr int BN = FUSED_UP ? 64 : 128;    // output columns per workgroup
};

__device__ __forceinline__ int chunk_at(int row, int c) { return row * ROW_BYTES + ((c ^ ((row >> 1) & 7)) * 16); }

// MF: activation fragments of 16 rows.  NJ: weight fragments per wavefront, 2 or, for half a tile's weight rows, 1 (gate+up:
// then 8 rows of each matrix, and the lanes of the upper half hold the up projection's sums).  SEG_K: the weights' K
// axis is cut in segments (shared experts' down projection), of any length.  Activation rows from a0 on, or those that `list` (LDS)
// names, or the tokens (g.sc_x) of the assignments that g.A names for the rows (an entry past the batch stands for the last token: no read outside
// the tokens).
enum class RowsFrom { HERE, LIST, ASSIGNMENTS };
template <bool FUSED_UP, bool SEG_K, int MF, int NJ, RowsFrom FROM>
__device__ __forceinline__ void tile_body(const GemmArgs &g, int slot, int m0, int m_end, int a0, int n0, int first_step,
                                          char *smem, const int16_t *list = nullptr) {
    constexpr int AHEAD = MF == 2 ? 8 : MF == 4 ? 6 : 4;   // steps in flight: what 256 registers hold (even)
    constexpr int AL = MF / 2;   // activation loads per thread and step: 32 rows each
    int tid = (int)threadIdx.x;
    asm volatile("" : "+v"(tid));   // what follows from it stays out of the kernel's loop over tiles
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, q = lane >> 4;
    const int nk = (g.K + BK - 1) / BK;

    // ---- load sources ----
    const auto a_rsrc = rsrc_of(FROM == RowsFrom::ASSIGNMENTS ? (const char *)g.sc_x : (const char *)g.A + (FROM == RowsFrom::HERE ? (int64_t)a0 * g.lda * 2 : 0));
    uint32_t a_off[AL];
    const int a_chunk = tid & 7;
#pragma unroll
    for (int i = 0; i < AL; ++i) {
        const int row = i * 32 + (tid >> 3);
        a_off[i] = NO_DATA;
        if (m0 + row < m_end) {
            const int from = FROM == RowsFrom::LIST ? list[row]
                             : FROM == RowsFrom::ASSIGNMENTS ? (int)min((uint32_t)((const int32_t *)g.A)[m0 + row] / (uint32_t)g.sc_k, (uint32_t)(g.sc_T - 1)) : row;
            a_off[i] = (uint32_t)from * (uint32_t)(g.lda * 2) + (uint32_t)a_chunk * 16u;
        }
    }
    const int wn = n0 + wave * (FUSED_UP ? 8 : 16) * NJ;   // first output column of the wavefront
    const int64_t b_first = ((int64_t)slot * g.b_slot_stride + (int64_t)wn * g.ldb) * 2;
    const auto b0_rsrc = rsrc_of((const char *)g.B0 + b_first);
    const auto b1_rsrc = rsrc_of((FUSED_UP ? (const char *)g.B1 : (const char *)g.B0) + b_first);
    // lane: row lane / 8 of every 8, 16-byte chunk lane % 8 (FUSED_UP: the first half of the rows gate, the second up)
    const int b_row = lane >> 3, b_chunk = lane & 7;
    uint32_t b_off[2 * NJ];
#pragma unroll
    for (int i = 0; i < 2 * NJ; ++i) {
        const int n = FUSED_UP ? (i % NJ) * 8 + b_row : i * 8 + b_row;
        b_off[i] = wn + n < g.N ? (uint32_t)n * (uint32_t)(g.ldb * 2) + (uint32_t)b_chunk * 16u : NO_DATA;
    }
    char *sb = smem + 2 * A_BYTES + wave * 2 * B_WAVE_BYTES;
    const int k_end = nk * BK;
    int bk = first_step * BK, b_left = nk;   // K of the next weight loads and how many there are (scalar)
    KSegWalk walk{b_chunk * 8};

    u32x4_t ra[AHEAD][AL], rb[AHEAD][2 * NJ];
    f32x4_t acc[MF][NJ];
#pragma unroll
    for (int i = 0; i < MF; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};

    int ak = first_step * BK, a_left = nk;   // the same for the activation loads
    auto load_a = [&](int set) {
        const uint32_t none = a_left > 0 && ak + a_chunk * 8 < g.K ? 0u : NO_DATA;
#pragma unroll
        for (int i = 0; i < AL; ++i) ra[set][i] = load16(a_rsrc, a_off[i] | none, (uint32_t)ak * 2u);
        --a_left;
        ak = ak + BK == k_end ? 0 : ak + BK;
    };
    auto store_a = [&](int set, int buf) {
#pragma unroll
        for (int i = 0; i < AL; ++i)
            *(u32x4_t *)(smem + buf * A_BYTES + chunk_at(i * 32 + (tid >> 3), a_chunk)) = ra[set][i];
    };
    auto load_b = [&](int set) {
        const int k = bk + b_chunk * 8;
        const uint32_t add = SEG_K ? walk.next(k, g.K, g.kseg_len, g.kseg_stride, BK) : b_left > 0 && k < g.K ? 0u : NO_DATA;
#pragma unroll
        for (int i = 0; i < 2 * NJ; ++i)
            rb[set][i] = load16(FUSED_UP && i >= NJ ? b1_rsrc : b0_rsrc, SEG_K ? offset_with(b_off[i], add) : b_off[i] | add, (uint32_t)bk * 2u);
        --b_left;
        bk = SEG_K || bk + BK != k_end ? bk + BK : 0;
    };
    auto store_b = [&](int set, int buf) {
#pragma unroll
        for (int i = 0; i < 2 * NJ; ++i) *(u32x4_t *)(sb + buf * B_WAVE_BYTES + chunk_at(i * 8 + b_row, b_chunk)) = rb[set][i];
    };
    // Two groups of 32 K.  The second group's fragments are read while the first is multiplied, each
    // activation fragment into the registers that its predecessor has just freed.
    bf16x8_t fa[MF], fb[2][NJ];
    auto read_b = [&](int gk, int buf) {
#pragma unroll
        for (int j = 0; j < NJ; ++j) fb[gk][j] = *(const bf16x8_t *)(sb + buf * B_WAVE_BYTES + chunk_at(j * 16 + r, gk * 4 + q));
    };
    auto read_a = [&](int i, int gk, int buf) { fa[i] = *(const bf16x8_t *)(smem + buf * A_BYTES + chunk_at(i * 16 + r, gk * 4 + q)); };
    auto mma = [&](int i, int gk) {
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[gk][j], fa[i], acc[i][j], 0, 0, 0);
    };
    auto compute = [&](int buf) {
        read_b(0, buf);
#pragma unroll
        for (int i = 0; i < MF; ++i) read_a(i, 0, buf);
        read_b(1, buf);
#pragma unroll
        for (int i = 0; i < MF; ++i) {
            mma(i, 0);
            read_a(i, 1, buf);
        }
#pragma unroll
        for (int i = 0; i < MF; ++i) mma(i, 1);
        __builtin_amdgcn_sched_group_barrier(0x100, MF + 2 * NJ, 0);   // LDS reads
#pragma unroll
        for (int i = 0; i < MF; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, NJ, 0);    // MFMA
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, NJ * MF, 0);
        __builtin_amdgcn_sched_barrier(0);
    };

    // ---- K loop: step s multiplies LDS buffer s % 2 with weight set s % AHEAD ----
    // The activation loads go out ahead of the weights': the wait for them at the end of the next step then leaves
    // that step's and the following one's weights in flight.
    auto step = [&](int p) {
        load_a(p % AHEAD);
        load_b(p);
        __builtin_amdgcn_sched_barrier(0);
        compute(p & 1);
        store_a((p + 1) % AHEAD, (p + 1) & 1);
        store_b((p + 1) % AHEAD, (p + 1) & 1);
        __syncthreads();
    };
#pragma unroll
    for (int p = 0; p < AHEAD; ++p) {
        load_a(p);
        load_b(p);
    }
    store_a(0, 0);
    store_b(0, 0);
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

    // ---- epilogue: element v of lane l of a block is output column 4 * (l / 16) + v, row l % 16 ----
    uint16_t *out = (uint16_t *)g.out;
#pragma unroll
    for (int i = 0; i < MF; ++i) {
        const int row = m0 + i * 16 + r;
        float up[4];
        if constexpr (FUSED_UP) {
#pragma unroll
            for (int v = 0; v < 4; ++v) up[v] = NJ == 2 ? acc[i][NJ - 1][v] : __shfl_xor(acc[i][0][v], 32, 64);
        }
        if (row >= m_end) continue;
#pragma unroll
        for (int j = 0; j < (FUSED_UP ? 1 : NJ); ++j) {
            const int col = wn + j * 16 + 4 * q;
            if (col >= g.N || (FUSED_UP && NJ == 1 && q >= 2)) continue;   // N is a multiple of 8
            float h[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                h[v] = acc[i][j][v];
                if (FUSED_UP) h[v] = h[v] * __frcp_rn(1.0f + __expf(-h[v])) * up[v];
            }
            *(uint2 *)(out + (int64_t)row * g.ldo + col) = make_uint2(pack_bf16x2(h[0], h[1]), pack_bf16x2(h[2], h[3]));
        }
    }
}

// Which of `count` numbers workgroup b works on, or -1: 64 runs of equal length, dealt to the XCDs in turn.
__device__ __forceinline__ int of_runs(int b, int count) {
    const int xcd = b & 7, j = b >> 3, len = (count + 63) >> 6, chunk = j / max(len, 1), t = (xcd + 8 * chunk) * len + (j - chunk * len);
    return chunk < 8 && t < count ? t : -1;
}

// Workgroups of the largest launch that `tiles` or fewer tiles make: the tiles, or one per compute unit and the others halved;
// few tiles are cut until there is about one per compute unit.  exact: there are that many.
inline int64_t grid_blocks(int64_t tiles, int n_cu, bool exact) {
    if (exact && 2 * tiles > 3 * (int64_t)n_cu) return (tiles + 63) / 64 * 64;
    const int64_t halves = std::min<int64_t>(2 * std::max<int64_t>(tiles - n_cu, 0), n_cu);
    return std::max((tiles + 63) / 64 * 64, (n_cu + 63) / 64 * 64 + (halves + 63) / 64 * 64);
}

// SEG_PER_LANE: 1 for up to 64 row segments, 4 for up to 256.  The grid covers the pieces of a rank with five times its share
// of the rows; what is more is walked in rounds, and what is less exits.  (A workgroup without work takes 1 to 1.5 us of a place for
// the segments' bounds: with one for every row of the batch, 3072 where 224 work, they took longer than the work, down
// projection of 591 rows in two segments, f = 352 15.9 us.)
//
// A compute unit has about 33 KB of loads in flight however many wavefronts ask, so one with two tiles takes twice as long as one
// with one, and with between one and two tiles per unit the launch lasts as long as two (alone 20 to 25 us, in pairs 32 to
// 38 us).  The tiles past one per unit are then cut in halves of 64 weight rows, a workgroup each.  Segments as a decode
// batch of 512 has them (16 segments, d = 2048, f = 1024, 1026 rows, 368 tiles), gate+up 36.7 -> 32.1 us, down 22.9 -> 20.2 us; 264
// tiles of f = 768 41.6 -> 32.3 us; shared experts' gate+up of 3001 rows, 352 tiles 36.0 -> 29.0 us.  Half tiles for all (672
// instead of 336) read the rows twice as often: 39.7 -> 39.9 us.  Up to one and a half tiles per unit, where tiles and halves still run
// all at once, two workgroups to a unit: shared experts' gate+up, whole -> halved, 384 tiles of d = 2048 34.5 -> 29.0 us, 396 33.6 ->
// 40.0 us, 432 34.0 -> 47.4 us, 448 of d = 4096 60.9 -> 82.7 us.
//
// Few tiles leave units without work, and a step's time falls with the bytes that its workgroup loads: up to one tile for every
// other unit all are halved (110 tiles, d = 2048, f = 1408, gate+up 22.5 -> 17.4 us, 80 tiles down 16.7 -> 12.3 us), and pieces are
// cut to 32 or 48 rows while there is a unit for each half (591 rows in two segments, f = 352, gate+up 22.5 -> 12.7 us; 64 rows
// of d = 4096, f = 14336, down 114 -> 60 us).  More halves than units are slower again (308 of 32 rows 16.0 us, 220 of 48 rows 15.0 us).
// With fewer than four steps along K there is too little to cut: K = 128, 64 tiles of 4 to 16 segments whole 5.5, halved 6.7 us (K = 256, 48
// tiles 7.0 -> 5.9 us).
// Rows to their positions: a row is read once and written k times, by one, two or four wavefronts (narrow rows by as many as have a piece of 64
// 16-byte vectors to move), AHEAD tokens at a time.  A token's positions wait in the lanes (64 at a time), so that no store waits for a load of its own.
// (With the workgroup per token narrow rows leave its wavefronts idle: layer steps of 97 tokens, k = 2, f = 352, d = 256, 512, 1024 45.0, 45.7, 32.8 -> 20.4,
// 21.6, 24.6 us.  Pieces dealt one by one are faster beside tiles whose weights come from HBM, 3001 tokens of d = 2048, f = 352, gate+up 56.9 -> 56.0 us, and
// slower beside weights in the last-level cache, 47.2 -> 50.0.)
constexpr int MOVE_AHEAD = 4;
__host__ __device__ inline int move_pieces(int row_bytes) { return (row_bytes + 1023) >> 10; }   // of a row
__device__ __forceinline__ void move_rows(const GemmArgs &g, int b, int movers) {
    const int vecs = g.sc_row_bytes >> 4, per_row = move_pieces(g.sc_row_bytes), n = g.sc_T * g.sc_k, lane = (int)threadIdx.x & 63;   // (n below 2^31)
    const int each_log = per_row >= 4 ? 2 : per_row == 2 ? 1 : 0;   // wavefronts of a token (three pieces: one after the other)
    const int first = (b << (2 - each_log)) + (__builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) >> each_log), step = movers << (2 - each_log);
    static_assert(THREADS == 256, "four wavefronts");
    const uint4 *const x = (const uint4 *)g.sc_x;
    uint4 *const xp = (uint4 *)g.sc_xp;
    for (int c0 = (int)threadIdx.x & ((64 << each_log) - 64); c0 < vecs; c0 += 64 << each_log) {   // whole wavefronts stay
        const int c = min(c0 + lane, vecs - 1);
        const bool store = c0 + lane < vecs;
        for (int t0 = first; t0 < g.sc_T; t0 += MOVE_AHEAD * step)
            for (int j0 = 0; j0 < g.sc_k; j0 += 64) {
                uint4 v[MOVE_AHEAD];
                int pos[MOVE_AHEAD];
#pragma unroll
                for (int i = 0; i < MOVE_AHEAD; ++i) {
                    const int64_t t = min(t0 + i * step, g.sc_T - 1);
                    v[i] = x[t * vecs + c];
                    pos[i] = g.sc_pos[t * g.sc_k + min(j0 + lane, g.sc_k - 1)];
                }
#pragma unroll
                for (int i = 0; i < MOVE_AHEAD; ++i) {
                    if (t0 + i * step >= g.sc_T) break;   // uniform
                    for (int j = 0; j < min(64, g.sc_k - j0); ++j) {
                        const int p = __builtin_amdgcn_readlane(pos[i], j);
                        if (p >= 0 && p < n && store) nt_store16(v[i], &xp[(int64_t)p * vecs + c]);
                    }
                }
            }
    }
}

// Workgroup number b of `grid` does its tiles.
template <bool FUSED_UP, bool SEG_K, int SEG_PER_LANE, RowsFrom FROM>
__device__ __forceinline__ void walk_tiles(const GemmArgs &g, int n_strips, int n_cu, int b, int grid, char *smem) {
    for (;;) {                              // once, unless the rank has far more rows than its share
        int lane = (int)threadIdx.x & 63;
        asm volatile("" : "+v"(lane));      // the table is read again each time: kept, it would cost the tile its registers
        SegTable<SEG_PER_LANE> segs;
        segs.load(g, lane);
        segs.cut(lane, BM);
        const bool few = g.K >= 4 * BK && 2 * segs.total * n_strips <= n_cu;
        if (few) {
            if (2 * segs.count(32) * n_strips <= n_cu) segs.cut(lane, 32);
            else if (2 * segs.count(48) * n_strips <= n_cu) segs.cut(lane, 48);
        }
        const int total = segs.total * n_strips, whole = few ? 0 : total > n_cu && 2 * total <= 3 * n_cu ? n_cu : total;
        const int whole_blocks = (whole + 63) & ~63, blocks = whole_blocks + ((2 * (total - whole) + 63) & ~63);
        if (b >= blocks) break;
        const int half = b < whole_blocks ? -1 : of_runs(b - whole_blocks, 2 * (total - whole));
        const int t = b < whole_blocks ? of_runs(b, whole) : half < 0 ? -1 : whole + half / 2;
        const bool again = b >= grid;
        b += grid;
        const bool more = b < blocks;
        if (t < 0) {
            if (more) continue;
            break;
        }
        const Segment s = segs.segment(t / n_strips, lane);
        const int in_seg = t - s.first_tile * n_strips, strip = in_seg / s.tiles, piece = in_seg - strip * s.tiles;
        const int rows = ((s.hi - s.lo + s.tiles - 1) / s.tiles + 15) & ~15;
        const int m0 = s.lo + piece * rows, m_end = min(s.hi, m0 + rows), a0 = FUSED_UP ? m0 : activation_row(g, s.slot, s.lo, m0);
        const int n0 = strip * Shape<FUSED_UP>::BN + (half < 0 ? 0 : (half & 1) * (Shape<FUSED_UP>::BN / 2));
        const int first_step = SEG_K ? 0 : (s.slot * n_strips + strip) / 4 % ((g.K + BK - 1) / BK);
        if (again) __syncthreads();   // the tile before has been read
        auto tile = [&](auto nj) {
            constexpr int NJ = decltype(nj)::value;
            if (m_end - m0 > 64) tile_body<FUSED_UP, SEG_K, 6, NJ, FROM>(g, s.slot, m0, m_end, a0, n0, first_step, smem);
            else if (m_end - m0 > 32) tile_body<FUSED_UP, SEG_K, 4, NJ, FROM>(g, s.slot, m0, m_end, a0, n0, first_step, smem);
            else if (m_end > m0) tile_body<FUSED_UP, SEG_K, 2, NJ, FROM>(g, s.slot, m0, m_end, a0, n0, first_step, smem);
        };
        if (half < 0) tile(std::integral_constant<int, 2>{});
        else if (n0 < g.N) tile(std::integral_constant<int, 1>{});
        if (!more) break;   // without reading the table once more (0.3 to 0.6 us of every launch)
    }
}

template <bool FUSED_UP, bool SEG_K, int SEG_PER_LANE>
__global__ __launch_bounds__(THREADS, 2) void gemm_bf16_mid_kernel(const GemmArgs g, int n_strips, int n_cu) {
    __shared__ __attribute__((aligned(1024))) char smem[LDS_BYTES];
    StaleRows stale;
    if (!FUSED_UP) stale = stale_rows(g);   // in flight during the work, used at the end
    walk_tiles<FUSED_UP, SEG_K, SEG_PER_LANE, RowsFrom::HERE>(g, n_strips, n_cu, (int)blockIdx.x, (int)gridDim.x, smem);
    if (FUSED_UP) share_record(g, blockIdx.x == 0); else clear_stale_rows(g, stale);
}

// Shared experts' and experts' projections in one launch, whose tiles run side by side: neither fills the chip by itself for all of its time, and
// one launch starts and ends once.  The gate+up launch also moves the dispatch rows: `movers` workgroups, ahead of the others, for which
// there are places beside the tiles; the experts' tiles read the tokens instead of the rows that are on their way.  Without shared
// experts (shared_blocks 0) it is the experts' projection and the rows.  Layer steps, a launch each -> joint, us, d = 2048: two shared experts, k = 6, f = 352,
// 97 tokens 54.7 -> 38.8, 800 68.0 -> 49.3, 3001 101.0 -> 80.8 (rows, shared and experts' gate+up 15.7 + 30 + 12, down 21 + 8.5); f = 1408, 400 tokens
// 85.1 -> 64.2; four shared experts, k = 4, f = 1408, 400 tokens 145.5 -> 126.2, only the down projections joint 800 184.5 -> 167.5; 1.24 times as fast in the
// mean of 27.  Without shared experts, k = 8, 512 tokens, f = 512 62.3 -> 59.0, 1000 80.5 -> 76.5; 37 steps of 97 to 3000 tokens 0.97 to 1.08, in the mean 1.033.
struct Joint {
    GemmArgs shared, experts;
    int shared_strips, expert_strips, shared_blocks, movers, n_cu;
};
template <bool FUSED_UP, int SEG_PER_LANE>
__global__ __launch_bounds__(THREADS, 2) void gemm_bf16_mid_joint_kernel(const Joint j) {
    __shared__ __attribute__((aligned(1024))) char smem[LDS_BYTES];
    StaleRows stale;
    if (!FUSED_UP) stale = stale_rows(j.experts);
    int b = (int)blockIdx.x;
    if (FUSED_UP && b < j.movers) {
        move_rows(j.experts, b, j.movers);
        return;
    }
    b -= j.movers;
    if (b < j.shared_blocks) {
        walk_tiles<FUSED_UP, !FUSED_UP, 1, RowsFrom::HERE>(j.shared, j.shared_strips, j.n_cu, b, j.shared_blocks, smem);
    } else {
        b -= j.shared_blocks;
        walk_tiles<FUSED_UP, false, SEG_PER_LANE, FUSED_UP ? RowsFrom::ASSIGNMENTS : RowsFrom::HERE>(
            j.experts, j.expert_strips, j.n_cu, b, (int)gridDim.x - j.movers - j.shared_blocks, smem);
        if (FUSED_UP) share_record(j.experts, b == 0);
    }
    if (!FUSED_UP) clear_stale_rows(j.experts, stale);
}

}  // namespace mid
}  // namespace grace
