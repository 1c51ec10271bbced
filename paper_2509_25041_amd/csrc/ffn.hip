// grace_expert_ffn / grace_shared_ffn: grouped SwiGLU FFN.
//
// Two grouped GEMM launches per call.  Operands are K-contiguous on both sides
// (activations [rows, K]; weights [N, K], one output feature per row), which is
// the layout the MFMA units consume directly:
//   up:   h[p, n]  = silu(sum_c xp[p,c] Wg[n,c]) * (sum_c xp[p,c] Wu[n,c])   K = d, N = f
//   down: y[p, m]  = sum_n h[p,n] Wd[m,n]                                     K = f, N = d
// Rows are grouped by instance: the rows of one rank are a contiguous range of
// the dispatch buffer, subdivided per local slot by inst_off (read on the
// device; there is no host synchronisation).  route_gemm below chooses the kernel
// by type, batch and shape.  The large-tile bf16 kernel is persistent (one
// workgroup per compute unit walks the tiles); the 96-row kernels launch for five times
// the rank's even share of the rows and walk what is more in rounds; the others size their
// grid from an upper bound of the tile count.  Surplus blocks exit at once.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "bf16.h"
#include "common.h"
#include "ffn_tiny.h"
#include "gemm_bf16_generic.h"
#include "gemm_bf16_mid.h"
#include "gemm_bf16_persist.h"
#include "gemm_common.h"
#include "gemm_f32.h"
#include "gemm_f32_split.h"
#include "gemm_stream.h"

namespace grace {

// Zeroes n 16-byte vectors (a kernel, not a memset: the call may be captured into a graph).
__global__ __launch_bounds__(256) void zero_fill_kernel(uint4 *__restrict__ out, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) out[i] = make_uint4(0u, 0u, 0u, 0u);
}

// Compute units of the current device (cached per device).
static int compute_units() {
    static int cached[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return -1;
    if (cached[dev] == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) return -1;
        cached[dev] = n;
    }
    return cached[dev];
}

// Dynamic LDS that a launch may ask for without opting in.  Kernels that take more (the persistent ones 160 KB) are opted in, once per kernel and
// device.
constexpr int LDS_WITHOUT_ASKING = 65536;
static bool allow_full_lds(const void *kernel, const char *what) {
    constexpr int MAX_KERNELS = 64, MAX_DEVICES = 64;
    static std::mutex mu;
    static const void *known[MAX_KERNELS] = {nullptr};
    static bool done[MAX_KERNELS][MAX_DEVICES] = {{false}};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) {
        fail(GRACE_EHIP, "%s: cannot query the device", what);
        return false;
    }
    std::lock_guard<std::mutex> lock(mu);
    int slot = 0;
    while (slot < MAX_KERNELS && known[slot] && known[slot] != kernel) ++slot;
    if (slot == MAX_KERNELS) {
        fail(GRACE_EHIP, "%s: kernel table full", what);
        return false;
    }
    known[slot] = kernel;
    if (!done[slot][dev]) {
        const hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, pers::LDS_BYTES);
        if (e != hipSuccess) {
            fail(GRACE_EHIP, "%s: cannot reserve LDS: %s", what, hipGetErrorString(e));
            return false;
        }
        done[slot][dev] = true;
    }
    return true;
}

// Can the kernels with buffer loads read these operands?  Rows of whole 16-byte vectors, K segments (where there are
// several) of a multiple of `kseg_align`, and offsets that fit (at most 128 rows are addressed from one base).
template <int EL>
static bool stream_ok(const GemmArgs &g, int kseg_align = strm::kstep<EL>()) {
    const int n_kseg = (g.K + g.kseg_len - 1) / g.kseg_len;
    const int64_t k_bytes = ((n_kseg - 1) * g.kseg_stride + g.kseg_len) * EL;
    return g.K % (16 / EL) == 0 && (n_kseg == 1 || g.kseg_len % kseg_align == 0) &&
           k_bytes + 128 * std::max(g.lda, g.ldb) * EL < (int64_t)NO_DATA;
}

// Which kernel takes a launch.
enum class Route {
    STREAM = GRACE_KERNEL_STREAM,
    MID = GRACE_KERNEL_MID,
    PERSIST = GRACE_KERNEL_PERSIST,
    GENERIC = GRACE_KERNEL_GENERIC,
    VECTOR_F32 = GRACE_KERNEL_VECTOR_F32,
};
// A rank hosts an expert at most once, so its row segments fit the kernels' segment tables.
static_assert(GRACE_MAX_EXPERTS <= pers::MAX_SEGMENTS, "more row segments than the kernels' tables hold");

// What the host knows of a launch's rows.
struct Rows {
    int max_rows;        // of one segment, as the callers' routing gives them (a token picks an expert once); more are still computed correctly
    int64_t picks;       // rows of all segments if the batch spreads evenly over the instances: picks / instances
    int instances;
    bool even_only;      // and that is what they are (all instances here, or one segment)
    int64_t most;        // bound on the rows of all segments that the routing gives
    int64_t m_bound;     // and whatever it gives

    // rows of all segments at `quarters` / 4 times the even share
    int64_t at(int quarters) const { return std::min(most, picks * quarters / (4 * (int64_t)instances)); }
};

struct Grid {
    int64_t groups;
    int threads;   // per workgroup
};
// Work-items of a launch along x have to fit 32 bits (HIP refuses more).
static bool launchable(const Grid &l) { return l.groups * l.threads <= (int64_t)UINT32_MAX; }

// fp32, more rows than one workgroup takes: workgroups per piece of the rows as well
template <int EL>
static bool stream_pieces(const Rows &rows) { return EL == 4 && rows.max_rows > strm::MAX_ROWS; }

// Streaming kernel.  With at most strm::MAX_ROWS rows per segment, one workgroup per strip of weight rows and
// segment.  At most one workgroup per strip and row of the batch finds work; with few of those each gets more
// than four wavefronts (a finer split of K) until the chip holds about 8 wavefronts per compute unit.  More than
// that does not pay (bf16, weights partly in the last-level cache): 16 per unit took 8.6 instead of 8.2 us on 4 busy
// segments, 32 took 10.4, and 32.9 instead of 28.8 us on 16; two wavefronts per workgroup at the other end took 29.5 us.
static int stream_fragments(const Rows &rows) { return rows.max_rows <= 16 ? 1 : rows.max_rows <= 32 ? 2 : 4; }
template <bool FUSED_UP, int EL>
static Grid stream_grid(const GemmArgs &g, const Rows &rows, int n_cu, int64_t others = 0 /* busy workgroups beside them */) {
    const int64_t n_strips = (g.N + strm::Shape<FUSED_UP>::COLS - 1) / strm::Shape<FUSED_UP>::COLS;
    if (stream_pieces<EL>(rows)) return {(std::max<int64_t>((rows.m_bound / strm::MAX_ROWS + g.S) * n_strips, n_cu) + 7) / 8 * 8, 256};
    const int64_t busy = std::min<int64_t>(g.S, rows.m_bound) * n_strips + others;
    int waves = 4;
    while (waves < strm::MAX_WAVES && strm::lds_bytes(waves * 2, stream_fragments(rows)) <= LDS_WITHOUT_ASKING &&
           busy * waves * 2 <= (int64_t)n_cu * 8 && g.K >= waves * 2 * 2 * strm::kstep<EL>())
        waves *= 2;
    return {n_strips * g.S, waves * 64};
}
template <bool FUSED_UP>
static Grid mid_grid(const GemmArgs &g, const Rows &rows, int n_cu) {
    const int64_t n_strips = (g.N + mid::Shape<FUSED_UP>::BN - 1) / mid::Shape<FUSED_UP>::BN;
    // ranks hold at most 4.9 times their instances' even share in the tables of the planner; the kernel walks in rounds what is more
    const int64_t expected = rows.even_only ? rows.m_bound : rows.at(20);
    const bool exact = g.M_single > 0;   // the shared experts
    return {mid::grid_blocks((exact ? (expected + mid::BM - 1) / mid::BM : expected / mid::BM + g.S) * n_strips, n_cu, exact), mid::THREADS};
}
// Tiles of the fp32 split kernel at `m` rows, a piece extra for every segment.
template <bool FUSED_UP>
static int64_t split_tiles(const GemmArgs &g, const Rows &rows, int64_t m) {
    constexpr int BN = split::Shape<FUSED_UP>::BN;
    return (m / split::BM + std::min<int64_t>(g.S, m)) * ((g.N + BN - 1) / BN);
}
// Groups of wavefronts that share a tile's K: two in down projections, whose K is long, while the tiles (half a piece extra for every segment)
// are one round of one per compute unit; with more, tiles run two to a unit.  Time with one group over time with two (median of 600 shared
// experts): up to a quarter of a round 1.33, to half 1.27, to one 1.11, to one and a half 0.91.  A rank's segments may make fewer tiles: K of 1024 or
// more, up to five quarters of a round 1.03 (0.92 to 1.24).
template <bool FUSED_UP>
static int split_groups(const GemmArgs &g, const Rows &rows, int n_cu) {
    if (FUSED_UP) return 1;
    const int64_t m = rows.at(4), strips = (g.N + split::Shape<false>::BN - 1) / split::Shape<false>::BN;
    if (g.S == 1) return (m + split::BM - 1) / split::BM * strips <= n_cu ? 2 : 1;
    const int64_t half_tiles = (2 * m / split::BM + std::min<int64_t>(g.S, m)) * strips;
    return 2 * half_tiles <= (g.K >= 1024 ? 5 : 4) * n_cu ? 2 : 1;
}
template <bool FUSED_UP>
static Grid split_grid(const GemmArgs &g, const Rows &rows, int n_cu) {
    const int64_t tiles = split_tiles<FUSED_UP>(g, rows, rows.even_only ? rows.m_bound : rows.at(20));
    const int groups = split_groups<FUSED_UP>(g, rows, n_cu);
    return {(std::max<int64_t>(tiles, 2 / groups * n_cu) + 63) / 64 * 64, 256 * groups};
}
// All tiles of the rows that a rank could hold, in whole runs of the XCDs, are one launch at most: their numbers fit 32 bits and so
// does every grid above (a hot rank's are walked by fewer workgroups).
template <bool FUSED_UP, typename SHAPE, int TILE_ROWS>
static bool mid_tiles_fit(const GemmArgs &g, const Rows &rows) {
    const int64_t n_strips = (g.N + SHAPE::BN - 1) / SHAPE::BN;
    return launchable({((rows.m_bound / TILE_ROWS + g.S) * n_strips + 63) / 64 * 64, mid::THREADS});
}
template <bool FUSED_UP>
static Grid grid_of(Route route, const GemmArgs &g, grace_dtype dt, const Rows &rows, int n_cu) {
    if (route == Route::STREAM)
        return dt == GRACE_BF16 ? stream_grid<FUSED_UP, 2>(g, rows, n_cu) : stream_grid<FUSED_UP, 4>(g, rows, n_cu);
    if (route == Route::MID) return dt == GRACE_BF16 ? mid_grid<FUSED_UP>(g, rows, n_cu) : split_grid<FUSED_UP>(g, rows, n_cu);
    if (route == Route::PERSIST) return {pers::grid_blocks(n_cu), pers::THREADS};
    if (route == Route::GENERIC) {
        constexpr int BN = FUSED_UP ? 64 : 128;
        return {(rows.m_bound / BM + g.S) * ((g.N + BN - 1) / BN), 256};
    }
    return {(rows.m_bound / FBM + g.S) * ((g.N + FBN - 1) / FBN), 256};
}

// Row pieces of at most bm rows that `rows` rows of up to n_seg segments make: ragged ends add quarters / 4 pieces to every
// segment that has rows.  Where most segments hold less than a piece the few hot ones still make hot / 4 of what all rows
// together would: a piece per segment may just fill the large kernel's rounds.
static int64_t pieces_of(int64_t rows, int n_seg, int bm, int quarters, int hot) {
    if (n_seg == 1) return (rows + bm - 1) / bm;
    const int64_t hit = std::max<int64_t>(1, std::min<int64_t>(n_seg, rows));
    return std::max(4 * hit * bm + hot * rows, 4 * rows + quarters * hit * bm) / (4 * bm);
}

// The 96-row kernel against 256 x 256 tiles.  The large tiles take their time by whole rounds over the compute units,
// however few rows a tile holds; the 96-row kernel by the number of its tiles.  With the rows of every segment known the line
// is sharp: gate+up, 2 x n_cu tiles while the large kernel needs one round and 3 x n_cu for every further round, down
// (where the large tiles adapt their height) about 2 and 2.6.  The host knows the rows for the shared experts, and their sum
// where a rank hosts all instances.  Elsewhere ranks hold 0.5 to 4.9 times their instances' even share in the tables of
// the planner.  At some loads the large tiles just fill their rounds, so the 96-row kernel is taken only if it is the
// cheaper one at the even share and at 7/4 (gate+up) or 3 times (down, where a wrong choice costs more) of it, and
// has at most 3 (gate+up) or 2 tiles per round and compute unit for a rank with three times its share.  Higher loads in the
// check lose more where ranks hold less than they save where one holds it (gate+up at 512 tokens, d = 2048, f = 1024: 50.7
// instead of 37.5 us with 9/4).
//
// Measured over 51204 projections inside 18287 layer steps (ranks of tables for five layer shapes, expert widths whole to a
// quarter, 1 to 32 ranks, 17 to 12000 tokens, three sets of weights in turn, the row scatter included where the large tiles
// carry it): 3008 ms with large tiles wherever they can run, 2178 with this rule and the one below, 2122 with the best kernel
// each time.  481 projections are slower than with large tiles by more than 3 % and 1 us, by 85 % at most (a rank with four times
// its share, 44.7 -> 82.8 us); of the steps, taking their projections together, 52 by more than 3 %, by 22 % at most.  The other way round the
// rule leaves 1556 projections on large tiles where 96 rows would be faster by as much, by 2.5 times at most: ranks with a tenth of
// their share (158 rows of 8963 tokens, 46.7 and 18.8 us), which the host cannot know.
template <bool FUSED_UP>
static bool mid_is_cheaper(const GemmArgs &g, const Rows &rows, int n_cu) {
    const int64_t strips = (g.N + mid::Shape<FUSED_UP>::BN - 1) / mid::Shape<FUSED_UP>::BN;
    const int64_t large_strips = (g.N + pers::Shape<FUSED_UP>::BN - 1) / pers::Shape<FUSED_UP>::BN;
    constexpr int HOT = FUSED_UP ? 1 : 0;   // (the down projection's large tiles get lower instead)
    const bool known = rows.even_only && g.S > 1;
    for (const int load : {4, FUSED_UP ? 7 : 12}) {   // quarters of the even share
        const int64_t m = rows.at(load);
        const int64_t tiles = pieces_of(m, g.S, mid::BM, FUSED_UP ? 2 : 3, HOT) * strips;
        const int64_t rounds = (pieces_of(m, g.S, pers::BM, 2, HOT) * large_strips + n_cu - 1) / n_cu;
        // in tenths of n_cu
        const int64_t limit = FUSED_UP ? 30 * rounds - (known ? 10 : 11) : 26 * rounds - 5;
        if (10 * tiles > n_cu * limit) return false;
        if (rows.even_only) break;
    }
    if (known) return true;
    // a rank that holds three times its share, with a whole piece extra for every segment
    const int64_t m = rows.at(12), hit = std::max<int64_t>(1, std::min<int64_t>(g.S, m));
    const int64_t rounds = ((m / pers::BM + hit) * large_strips + n_cu - 1) / n_cu;
    return (m / mid::BM + hit) * strips <= n_cu * rounds * (FUSED_UP ? 3 : 2);
}

// fp32, batches of more than 64 tokens: the split kernel (MID) against the streaming one, whose pieces of 64 rows and 32 weight rows make
// eight times as many workgroups and whose wavefronts share K.  Few tiles, short K and segments of a few rows each, whose weights are all
// that there is to move, are for that one.  The host knows the rows of the shared experts and of a rank that hosts all instances, elsewhere
// their even share.
//
// Measured over 1889 gate+up and as many down projections (1289 of experts: 15 sizes from 128 x 256 to 4096 x 512, 768 x 3072 and 2048 x 2048, 548
// and 1388 among them, 1 to 128 segments on 1 to 4 ranks, even to Zipf-shaped shares, 65 to 5000 tokens, k = 1, 2 and 8; 600 of one
// to four shared experts), weights of 700 MB or more in turn, each kernel alone:
//   gate+up: streaming 296.5 ms, split 194.3, this rule 192.8, the better one each time 191.8;
//   down: streaming 164.1, split 132.0 (one group) and 127.7 (two), this rule 119.8, the best one each time 117.6.
// With the fp32 matrix instruction alone (streamed, or 96 x 64 tiles where they were faster) they took 268.4 and 159.2; 246 of the 3778 are slower than
// that by more than 3 %, 64 by more than 10 %, by 47 % at most: ranks that hold far fewer rows than their share, and segments of a few rows.
template <bool FUSED_UP>
static bool split_is_faster(const GemmArgs &g, const Rows &rows, int n_cu) {
    const int64_t m = rows.at(4), segments = std::min<int64_t>(g.S, std::max<int64_t>(m, 1));
    const int64_t percent = 100 * split_tiles<FUSED_UP>(g, rows, m) / n_cu;   // tiles per compute unit
    if constexpr (FUSED_UP) {
        if (m <= 3 * segments) return percent >= 500;
        return percent >= (g.K >= 512 ? 42 : g.K >= 192 ? 70 : 125);
    } else {
        // (rows of a segment times K: what its weights, of whatever width, are multiplied with)
        if (split_groups<false>(g, rows, n_cu) == 2) return percent >= 30 && g.K >= 512 && m * g.K > (percent >= 50 ? 8000 : 16000) * segments;
        return percent > 400 || m * g.K > 6000 * segments;
    }
}

// bf16, up to 64 rows per segment: the streaming kernel, which splits the work finest, while the 96-row kernel's tiles
// would not fill the chip.  A gate+up projection of more than 16 rows leaves it when the other has a tile for three quarters
// of the compute units, a down projection when there are one and a half per unit, and with few steps along K only past 32
// tokens (21 tokens, d = 2048, f = 384, 128 segments 11.4 us, 14.2 with the other).  Time of the streaming kernel over that of the 96-row
// kernel in the steps above with 17 to 64 tokens (median, and what 96 of 100 lie between), by tiles per compute unit at three times the even share:
//   gate+up: up to 1/4 0.86 (0.71 to 1.17), to 3/4 1.12 (0.74 to 1.59), to 1 1.29 (0.97 to 1.73), to 3/2 1.44 (1.21 to 1.97), more 1.21 (1.02 to 1.48)
//   down, K >= 1024: up to 1/4 0.91 (0.71 to 1.28), to 1 1.09 (0.78 to 1.36), to 3/2 1.16 (1.02 to 1.34), more 1.30 (1.05 to 1.63)
//   down, K < 1024: up to 1 0.89 (0.74 to 1.09), to 3/2 0.96 (0.83 to 1.31), more 1.15 (0.99 to 1.38)
// All 8257 such gate+up projections take 281.6 ms with the streaming kernel, 235.0 with 96 rows, 237.4 with this rule and 229.7
// with the best kernel each time; the down projections 188.1, 177.9, 179.7 and 169.0.
template <bool FUSED_UP>
static Route route_gemm(const GemmArgs &g, grace_dtype dt, const Rows &rows, int n_cu) {
    auto fits = [&](Route r) { return launchable(grid_of<FUSED_UP>(r, g, dt, rows, n_cu)); };
    if (dt == GRACE_F32) {
        const bool stream = stream_ok<4>(g) && fits(Route::STREAM);
        // K segments of any length (shared experts' down projection, f = 1388, two of them, d = 1024, 65 to 5000 tokens: vector ALUs
        // 329 to 577 us, with 96 x 64 tiles of the fp32 instruction 38 to 289)
        const bool split = stream_pieces<4>(rows) && stream_ok<4>(g, 4) && mid_tiles_fit<FUSED_UP, split::Shape<FUSED_UP>, split::BM>(g, rows);
        if (split && (!stream || split_is_faster<FUSED_UP>(g, rows, n_cu))) return Route::MID;
        return stream ? Route::STREAM : Route::VECTOR_F32;
    }
    const bool mid_ok = stream_ok<2>(g, 8) && mid_tiles_fit<FUSED_UP, mid::Shape<FUSED_UP>, mid::BM>(g, rows);
    if (rows.max_rows <= strm::MAX_ROWS && stream_ok<2>(g) && fits(Route::STREAM)) {
        const int64_t busy = std::max<int64_t>(1, std::min<int64_t>(g.S, rows.at(12)));
        const int64_t tiles = busy * ((g.N + mid::Shape<FUSED_UP>::BN - 1) / mid::Shape<FUSED_UP>::BN);
        if (!mid_ok || rows.max_rows <= 16 || tiles <= (FUSED_UP ? n_cu * 3 / 4 : n_cu * 3 / 2)) return Route::STREAM;
        if (!FUSED_UP) return rows.max_rows > 32 || g.K >= 1024 ? Route::MID : Route::STREAM;
    }
    const bool persist_ok = g.K % pers::BK == 0 && g.kseg_len % pers::BK == 0 && g.K >= pers::MIN_K_STEPS * pers::BK;
    if (!mid_ok) return persist_ok ? Route::PERSIST : Route::GENERIC;
    return !persist_ok || mid_is_cheaper<FUSED_UP>(g, rows, n_cu) ? Route::MID : Route::PERSIST;
}

template <bool FUSED_UP, int EL>
static void launch_stream(const GemmArgs &g, const Rows &rows, const Grid &l, int n_cu, hipStream_t st) {
    const int n_strips = (g.N + strm::Shape<FUSED_UP>::COLS - 1) / strm::Shape<FUSED_UP>::COLS;
    if constexpr (EL == 4) {
        if (stream_pieces<EL>(rows)) {
            const int lds = strm::lds_bytes(4, strm::MAX_ROWS / 16);
            if (g.S <= 64) strm::gemm_stream_tiles_kernel<FUSED_UP, EL, 1><<<(unsigned)l.groups, l.threads, lds, st>>>(g, n_strips, n_cu);
            else strm::gemm_stream_tiles_kernel<FUSED_UP, EL, 4><<<(unsigned)l.groups, l.threads, lds, st>>>(g, n_strips, n_cu);
            return;
        }
    }
    auto launch = [&](auto mf) {
        constexpr int MF = decltype(mf)::value;
        strm::gemm_stream_kernel<FUSED_UP, EL, MF><<<(unsigned)l.groups, l.threads, strm::lds_bytes(l.threads / 64, MF), st>>>(g, n_strips);
    };
    const int mf = stream_fragments(rows);
    if (mf == 1) launch(std::integral_constant<int, 1>{});
    else if (mf == 2) launch(std::integral_constant<int, 2>{});
    else launch(std::integral_constant<int, 4>{});
}

template <bool FUSED_UP>
static int launch_split(const GemmArgs &g, const Grid &l, int n_cu, hipStream_t st, const char *what) {
    const int groups = l.threads / 256;
    const void *kernel = FUSED_UP ? split::up_kernel() : g.kseg_len < g.K ? split::shared_down_kernel(groups) : split::down_kernel(groups);
    if (!allow_full_lds(kernel, what)) return GRACE_EHIP;
    GemmArgs args = g;
    int n_strips = (g.N + split::Shape<FUSED_UP>::BN - 1) / split::Shape<FUSED_UP>::BN;
    void *params[] = {&args, &n_strips, &n_cu};
    (void)hipLaunchKernel(kernel, dim3((unsigned)l.groups), dim3(l.threads), params, groups * split::GROUP_BYTES, st);   // (the caller asks for the error)
    return GRACE_OK;
}

template <bool FUSED_UP>
static void launch_mid(const GemmArgs &g, const Grid &l, int n_cu, hipStream_t st) {
    const int n_strips = (g.N + mid::Shape<FUSED_UP>::BN - 1) / mid::Shape<FUSED_UP>::BN;
    if constexpr (!FUSED_UP) {   // K segments: the shared experts' down projection alone
        if (g.kseg_len < g.K) {
            mid::gemm_bf16_mid_kernel<false, true, 1><<<(unsigned)l.groups, l.threads, 0, st>>>(g, n_strips, n_cu);
            return;
        }
    }
    if (g.S <= 64) mid::gemm_bf16_mid_kernel<FUSED_UP, false, 1><<<(unsigned)l.groups, l.threads, 0, st>>>(g, n_strips, n_cu);
    else mid::gemm_bf16_mid_kernel<FUSED_UP, false, 4><<<(unsigned)l.groups, l.threads, 0, st>>>(g, n_strips, n_cu);
}

template <bool FUSED_UP, pers::Who WHO>
static int launch_gemm(const GemmArgs &g, grace_dtype dt, const Rows &rows, hipStream_t st, const char *what) {
    if (rows.m_bound <= 0 || g.N <= 0 || g.K <= 0) return GRACE_OK;
    const int n_cu = compute_units();
    if (n_cu <= 0) return fail(GRACE_EHIP, "%s: cannot query the device", what);
    const Route route = route_gemm<FUSED_UP>(g, dt, rows, n_cu);
    const Grid l = grid_of<FUSED_UP>(route, g, dt, rows, n_cu);
    if (!launchable(l)) return fail(GRACE_ESHAPE, "%s: grid too large", what);
    if (route == Route::STREAM) {
        if (dt == GRACE_BF16) launch_stream<FUSED_UP, 2>(g, rows, l, n_cu, st);
        else launch_stream<FUSED_UP, 4>(g, rows, l, n_cu, st);
    } else if (route == Route::MID && dt == GRACE_F32) {
        const int rc = launch_split<FUSED_UP>(g, l, n_cu, st, what);
        if (rc != GRACE_OK) return rc;
    } else if (route == Route::MID) {
        launch_mid<FUSED_UP>(g, l, n_cu, st);
    } else if (route == Route::PERSIST) {
        // persistent large-tile kernel: one workgroup per compute unit, 160 KB of dynamic LDS
        using SH = pers::Shape<FUSED_UP>;
        const int ntn = (g.N + SH::BN - 1) / SH::BN;
        if ((rows.m_bound / 160 + g.S) * (int64_t)ntn > INT32_MAX) return fail(GRACE_ESHAPE, "%s: too many tiles", what);   // the lowest m-tile has 160 rows
        if (g.S <= 64) {
            if (!allow_full_lds((const void *)pers::gemm_bf16_persist_kernel<FUSED_UP, 1, WHO>, what)) return GRACE_EHIP;
            pers::gemm_bf16_persist_kernel<FUSED_UP, 1, WHO><<<(unsigned)l.groups, l.threads, pers::LDS_BYTES, st>>>(g, ntn);
        } else if constexpr (WHO != pers::SHARED) {  // the shared experts are a single row segment
            if (!allow_full_lds((const void *)pers::gemm_bf16_persist_kernel<FUSED_UP, 4, WHO>, what)) return GRACE_EHIP;
            pers::gemm_bf16_persist_kernel<FUSED_UP, 4, WHO><<<(unsigned)l.groups, l.threads, pers::LDS_BYTES, st>>>(g, ntn);
        }
    } else if (route == Route::GENERIC) {
        constexpr int BN = FUSED_UP ? 64 : 128;
        gemm_bf16_kernel<FUSED_UP><<<(unsigned)l.groups, l.threads, 0, st>>>(g, (g.N + BN - 1) / BN);
    } else {
        gemm_f32_kernel<FUSED_UP><<<(unsigned)l.groups, l.threads, 0, st>>>(g, (g.N + FBN - 1) / FBN);
    }
    GRACE_LAUNCH_CHECK(what);
    return GRACE_OK;
}

// Shared experts' and experts' projections as one launch of the 96-row kernel, where it takes both (gemm_bf16_mid_joint_kernel).
template <bool FUSED_UP>
static int launch_joint(const GemmArgs *shared, const Rows &shared_rows, const GemmArgs &experts, const Rows &rows, int n_cu, hipStream_t st, const char *what) {
    mid::Joint j{};
    const Grid e = grid_of<FUSED_UP>(Route::MID, experts, GRACE_BF16, rows, n_cu);
    int64_t tiles = 0;
    if (shared) {
        j.shared = *shared;
        j.shared_strips = (shared->N + mid::Shape<FUSED_UP>::BN - 1) / mid::Shape<FUSED_UP>::BN;
        tiles = (shared_rows.m_bound + mid::BM - 1) / mid::BM * j.shared_strips;
        j.shared_blocks = (int)mid::grid_blocks(tiles, n_cu, true);
    }
    j.experts = experts;
    j.expert_strips = (experts.N + mid::Shape<FUSED_UP>::BN - 1) / mid::Shape<FUSED_UP>::BN;
    j.n_cu = n_cu;
    if (FUSED_UP && experts.sc_T > 0) {
        // One round of loads per wavefront and 300 KB per workgroup at most, up to one for each compute unit: a round of pieces takes several us
        // whatever it moves, and short launches have no more.  d = 2048: 200 and 400 KB are even with 300, 800 slower where the rows are many (3001 tokens,
        // k = 6, f = 352 79.8, 80.8 and 87.0 us a step), and so are half as many workgroups at most (89.0).  Layer steps, any number of rounds -> four -> two ->
        // one: 512 tokens, k = 4, f = 352, two shared experts 51.5 -> 51.6 -> 49.3 -> 47.6 us; d = 256, 97 tokens, k = 2, f = 352, none 23.5 -> 20.4 -> 20.4 -> 20.4;
        // 207 steps (d = 256 to 4096, 97 to 3000 tokens) with one round 3 % faster in the mean than with any number, 0.4 % than with four.
        const int64_t bytes = (int64_t)experts.sc_T * (1 + experts.sc_k) * experts.sc_row_bytes;
        const int64_t pieces = (int64_t)experts.sc_T * mid::move_pieces(experts.sc_row_bytes), round = mid::MOVE_AHEAD * (mid::THREADS / 64);
        j.movers = (int)std::min<int64_t>(n_cu, std::max(bytes / (300 << 10) + 1, (pieces + round - 1) / round));
    }
    const Grid l = {j.movers + j.shared_blocks + e.groups, mid::THREADS};
    if (!launchable(l)) return fail(GRACE_ESHAPE, "%s: grid too large", what);
    if (experts.S <= 64) mid::gemm_bf16_mid_joint_kernel<FUSED_UP, 1><<<(unsigned)l.groups, l.threads, 0, st>>>(j);
    else mid::gemm_bf16_mid_joint_kernel<FUSED_UP, 4><<<(unsigned)l.groups, l.threads, 0, st>>>(j);
    GRACE_LAUNCH_CHECK(what);
    return GRACE_OK;
}

// Shapes of the two projections (operands are filled in by the entry points).
//   up:   K = d, N = f, two weight matrices        down: K = f, N = d
static GemmArgs expert_shape(bool up, int S, int d, int f) {
    GemmArgs g{};
    g.K = up ? d : f;
    g.N = up ? f : d;
    g.lda = g.ldb = g.kseg_len = g.K;
    g.ldo = g.N;
    g.b_slot_stride = (int64_t)d * f;
    g.S = S;
    return g;
}

// The shared experts act as one expert of width F = n_shared * f: gate and up weights [n_shared, f, d]
// are one [F, d] matrix each; the down weights [n_shared, d, f] are F input features in n_shared
// K segments of length f that lie d * f elements apart.
static GemmArgs shared_shape(bool up, int T, int d, int f, int n_shared) {
    GemmArgs g = expert_shape(up, 1, d, n_shared * f);
    g.b_slot_stride = 0;
    g.M_single = T;
    if (!up) {
        g.ldb = g.kseg_len = f;
        g.kseg_stride = (int64_t)d * f;
    }
    return g;
}

// Rows of a rank that hosts S of I instances, at most every token once per instance or choice.
static Rows expert_rows(int S, int I, int32_t T, int32_t k) {
    return {T, (int64_t)T * k * S, I, S == I, (int64_t)T * std::min(S, k), (int64_t)T * k};
}
static Rows shared_rows(int32_t T) { return {T, T, 1, true, T, T}; }

// Whether the joined gate+up projection is dealt out in units of 4 columns (ffn_tiny_cols.hip) rather than a workgroup per slot and strip (ffn_tiny.hip):
// up to 8 tokens, K in whole 128-byte lines.  Every workgroup waits for the whole gate then, which pays where slots without rows would leave
// workgroups idle: not for one or two slots (d = 4096, f = 3584, 1 to 8 tokens 0.91 to 1.04 times as fast), for more than 4 tokens not where a
// slot has fewer units than half the compute units (f = 192 and 256, 5 and 8 tokens 0.97 to 1.06), and not with shared experts, whose tiles
// need not wait (2 and 4 of f = 352 and 1408 0.88 to 1.05).  Where it is taken, steps of 1 to 8 tokens, 8 to 19 slots: f = 704 to 2816 1.01 to
// 1.21, in the mean 1.08; f = 192 and 256, up to 4 tokens 1.05 to 1.22.
static bool deals_columns(int S, int32_t T, int32_t d, int32_t f, grace_dtype dt, int n_cu) {
    return S > 2 && T <= TINY_COLS_T && (T <= 4 || f >= 2 * n_cu) && (int64_t)d * (dt == GRACE_F32 ? 4 : 2) % 128 == 0;
}

// One launch for the down projections and the combine of a joined step (ffn_tiny_down.hip): its operands fit 32-bit offsets and its partial
// sums the LDS.  A workgroup has 8 or 16 columns of everything to do, so narrow tokens leave compute units idle: with fewer
// workgroups than 5 for 8 of them it has to be little work each, and more of it where shared experts' own launch goes too.
// Whole steps, two or three launches -> one, bf16 | fp32, 2 to 16 tokens, rank with half the experts: d >= 1536 1.01 to 1.46 | 0.98 to 1.40 times
// as fast (f = 1024 to 4096; with 2 shared experts 1.01 to 1.35 | 1.00 to 1.31); d = 1024 with 4 parts 1.09 to 1.24 | 1.08 to 1.25, with 8 to 32
// 0.90 to 1.07 | 0.87 to 1.08; d = 512 with 4 1.12 to 1.20 | 1.14 to 1.25, with 8 to 32 0.77 to 0.97 | 0.75 to 0.92; with 2 shared
// experts and 10 to 18 parts d = 1024 1.13 to 1.38 | 1.09 to 1.34, d = 512 1.02 to 1.36 | 0.95 to 1.29.
static bool joins_combine(int32_t T, int32_t k, int32_t d, int32_t f, int n_shared, int S, grace_dtype dt, int n_cu) {
    const int64_t row = (int64_t)f * (dt == GRACE_F32 ? 4 : 2);
    if (T > TINY_DOWN_T || k > GRACE_MAX_TOPK || row % 16 != 0 || 16 * row >= (int64_t)NO_DATA || std::max(n_shared, 1) * T * row >= (int64_t)NO_DATA) return false;
    if (tiny_down_lds(T, k, S, n_shared, d, n_cu) > pers::LDS_BYTES) return false;
    const int blocks = tiny_down_blocks(d, n_cu), parts = std::min(S, T * k) + n_shared;
    return 8 * blocks >= 5 * n_cu || parts <= (n_shared ? std::max(16, blocks / 4) : 4);
}

// Whether tiny_up_kernel is faster than the two launches with `tiles` workgroups for the projection.  Every one of them looks for its rows (1.5 us), those
// of slots without rows too, which the projection's own launch leaves at once.  Layer steps, two launches -> joined, 700 drawn ones (d = 64 to 4096, f = 64 to
// 3584, 1 to 128 slots), by workgroups per compute unit, mean (least) times as fast: 9 to 32 tokens, bf16, up to 4 1.3 (1.02), 8 1.2 (1.03), 12 1.15 (1.01), 16
// 1.03 (0.91), 32 0.95 (0.82), 112 0.66 (118 instead of 74 us); fp32 up to 4 1.2 (1.04), 6 1.15 (0.95), 8 1.03 (0.91), 24 0.93 (0.82); up to 8 tokens with
// shared experts up to 24 1.3 (1.03), 64 0.94 (0.77), where the combine is joined too up to 44 1.4 (1.04), 64 1.0 (0.91).
// Pieces of 64 rows (fp32), more than 16 experts: the dispatch's workgroups have little less to do than a launch of their own, so it pays where all are resident at
// once (joined_waves: two per compute unit), 0.96 to 1.24, beyond 0.67 to 0.95; rows of 4 KB and more up to one per compute unit, which the launcher still cuts
// lower, 0.98 to 1.30 (219 tokens of 16 experts, d = 1536, f = 704, 352 pieces 43 -> 52 us).  Narrow rows and many choices of many experts likewise: beyond 0.89 to 0.98.
static bool tiny_up_pays(int64_t tiles, bool pieces, int32_t T, int32_t k, int32_t d, int32_t f, int E, int S, int n_shared, grace_dtype dt, int n_cu) {
    const int64_t row_bytes = (int64_t)d * (dt == GRACE_F32 ? 4 : 2);
    const int64_t most = pieces ? (row_bytes >= 4096 ? 1 : 2) : T > 32 ? 4 : T > 8 ? (dt == GRACE_BF16 ? 12 : 6) : joins_combine(T, k, d, f, n_shared, S, dt, n_cu) ? 56 : 24;
    if (tiles > most * n_cu) return false;
    if ((pieces && E > TINY_LANE_E) || (row_bytes <= 512 && E > 64 && T * k > 120)) return T + tiles <= 2 * (int64_t)n_cu;
    return true;
}

// Wavefronts per workgroup of tiny_up_kernel, `waves` by the tiles alone: where these are few and short, the dispatch's workgroups, which have as
// many, are the launch's end.  As many more as all workgroups can be resident with (16 wavefronts per compute unit).  Layer steps with `waves` = 4 -> 8 or 16,
// us: 128 experts, k = 8, d = 64, f = 352, 30 tokens 22.0 -> 16.1 (two launches 18.1), 64, d = 256, f = 512, 63 tokens 22.7 -> 18.4 (21.0); fp32, 64, k = 6, f = 512,
// 77 tokens 25.8 -> 21.4 (24.2).  Rows of more than 1 KB 0.97 to 1.09.
static int joined_waves(int waves, int64_t tiles, bool pieces, int32_t T, int32_t k, int32_t d, int E, grace_dtype dt, int n_cu) {
    if (E <= TINY_LANE_E || (!pieces && (int64_t)d * (dt == GRACE_F32 ? 4 : 2) > 1024)) return waves;
    const int most = T > 32 ? 8 : strm::MAX_WAVES, at_once = E <= 64 ? 4 : 1;   // tokens of the gate per wavefront
    while (waves < most && (waves * at_once < T || waves * 64 < T * k) && (T + tiles) * waves * 2 <= (int64_t)n_cu * 16) waves *= 2;
    return waves;
}

// Smallest batches: one launch for the dispatch and the experts' gate+up projection (ffn_tiny.hip), whose hidden activation the down
// projection then finds slot by slot.
static bool joins_dispatch(const grace_table *table, int32_t rank, int32_t T, int32_t k, int32_t d, int32_t f, int n_shared, grace_dtype dt, int n_cu) {
    const int S = table->rank_ptr[rank + 1] - table->rank_ptr[rank], el = dt == GRACE_F32 ? 4 : 2;
    if (S < 1 || !tiny_batch(T, k, table->E, table->I)) return false;
    if (S > k && (size_t)T * S * f * el > SLOT_ROWS_MOST) return false;
    const GemmArgs up = expert_shape(true, S, d, f), dn = expert_shape(false, S, d, f);
    const Rows rows = expert_rows(S, table->I, T, k);
    if ((up.K + T * up.lda) * el >= (int64_t)NO_DATA) return false;   // offsets of any token from the first
    const Route r = route_gemm<false>(dn, dt, rows, n_cu);
    if (r != Route::STREAM && !(r == Route::MID && dt == GRACE_BF16)) return false;
    const Route u = route_gemm<true>(up, dt, rows, n_cu);
    Grid l = grid_of<true>(u, up, dt, rows, n_cu);
    if (u == Route::MID && dt == GRACE_BF16) {
        if (T > mid::BM) return false;   // one piece per slot
        // (four wavefronts' dispatch is longer than the tiles: d = 256, 89 tokens of 60 experts, k = 6 24.8 -> 27.7 us a step, of 64, k = 8 37.1 -> 40.7)
        if ((int64_t)d * el <= 512 && table->E > TINY_LANE_E && T * k > 256) return false;
        l.groups = tiny_up_mid_blocks(S, up.K, (up.N + mid::Shape<true>::BN - 1) / mid::Shape<true>::BN, n_cu);
        if (l.groups == 0) return false;
    } else if (u == Route::STREAM) {
        const bool pieces = stream_pieces<4>(rows) && dt == GRACE_F32;
        l.groups = (int64_t)S * ((up.N + strm::Shape<true>::COLS - 1) / strm::Shape<true>::COLS) * (pieces ? (T + strm::MAX_ROWS - 1) / strm::MAX_ROWS : 1);
        const bool dealt = n_shared == 0 && deals_columns(S, T, d, f, dt, n_cu);
        if (!dealt && !tiny_up_pays(l.groups, pieces, T, k, d, f, table->E, S, n_shared, dt, n_cu)) return false;
    } else {
        return false;
    }
    l.groups += T + 8;
    l.threads = 64 * strm::MAX_WAVES;
    return launchable(l);
}

// Is a projection of the experts one launch with the shared experts' (n_shared > 0), or with the rows (n_shared == 0, gate+up)?  Offsets of the
// tokens that the gate+up tiles read fit 32 bits.
static bool joins_shared(bool up, int32_t T, int32_t k, int32_t d, int32_t f, int n_shared, int S, int I, grace_dtype dt, int n_cu) {
    if (dt != GRACE_BF16 || S < 1 || T < 1 || (int64_t)T * d * 2 >= (int64_t)NO_DATA || (int64_t)n_shared * f > INT32_MAX) return false;
    const Rows rows = expert_rows(S, I, T, k);
    if ((up ? route_gemm<true>(expert_shape(true, S, d, f), dt, rows, n_cu) : route_gemm<false>(expert_shape(false, S, d, f), dt, rows, n_cu)) != Route::MID) return false;
    if (n_shared == 0) return up && (S > 1 || T > 256);   // (one slot, d = 4096, k = 2: 97 and 200 tokens 0.97 to 1.01, 512 and 1000 1.02 to 1.04)
    const Rows all = shared_rows(T);
    return (up ? route_gemm<true>(shared_shape(true, T, d, f, n_shared), dt, all, n_cu)
               : route_gemm<false>(shared_shape(false, T, d, f, n_shared), dt, all, n_cu)) == Route::MID;
}

static int check_ffn_shapes(const char *who, int32_t d, int32_t f, grace_dtype dt) {
    if (dt != GRACE_F32 && dt != GRACE_BF16) return fail(GRACE_EINVAL, "%s: unknown dtype %d", who, (int)dt);
    if (d < 1 || f < 1) return fail(GRACE_EINVAL, "%s: d=%d, f=%d invalid", who, d, f);
    if (dt == GRACE_BF16 && ((d % 8) || (f % 8)))
        return fail(GRACE_ESHAPE, "%s: bf16 needs d and f to be multiples of 8 (d=%d, f=%d)", who, d, f);
    return GRACE_OK;
}

}  // namespace grace

using namespace grace;

static int expert_ffn_common(const char *who, const grace_table *table, int32_t rank, int32_t T, int32_t k, int32_t d,
                             int32_t f, grace_dtype dt, int &g0, int &S) {
    if (!table) return fail(GRACE_EINVAL, "%s: table is null", who);
    if (rank < 0 || rank >= table->R) return fail(GRACE_EINVAL, "%s: rank=%d outside [0,%d)", who, rank, table->R);
    if (T < 0 || k < 1) return fail(GRACE_EINVAL, "%s: T=%d, k=%d invalid", who, T, k);
    if ((int64_t)T * k > INT32_MAX) return fail(GRACE_ESHAPE, "%s: T*k exceeds 2^31-1", who);
    int rc = check_ffn_shapes(who, d, f, dt);
    if (rc != GRACE_OK) return rc;
    g0 = table->rank_ptr[rank];
    S = table->rank_ptr[rank + 1] - g0;
    return GRACE_OK;
}

static int shared_ffn_common(const char *who, int32_t T, int32_t d, int32_t f, int32_t n_shared, grace_dtype dt);

// Does the launch of a gate+up projection move the dispatch rows as well?  The large-tile kernel does, rows in whole 1 KB pieces of
// which a wavefront holds one with the positions of its token, a lane each (up to 64 choices); offsets of positions in 32 bits, and piece
// numbers (a wavefront looks at four strides of the grid at a time) below 2^31.  The experts' projection reads the tokens themselves then: their
// offsets fit 32 bits, and the rows of the next tile are looked up while three steps along K or more run.
static bool carries_rows(Route route, grace_dtype dt, int32_t T, int32_t k, int32_t d, bool experts) {
    const int64_t row_bytes = (int64_t)d * 2;
    if (route != Route::PERSIST || dt != GRACE_BF16 || row_bytes % 1024 != 0 || row_bytes > INT32_MAX) return false;
    if (k > 64 || (int64_t)T * k >= ((int64_t)1 << 29) || T * (row_bytes / 1024) > ((int64_t)1 << 30)) return false;
    return !experts || (d >= 3 * pers::BK && T * row_bytes <= (int64_t)INT32_MAX);
}

// Row scatter that a projection is to do as well: xp[pos[a]] = x[a / k]; src is the inverse of pos.
struct Scatter {
    const void *x;
    const int32_t *pos, *src;
};

static int expert_ffn_up(const char *who, const grace_table *table, int32_t rank, const void *xp, const int32_t *inst_off,
                         int32_t T, int32_t k, int32_t d, int32_t f, grace_dtype dt, const void *w_gate, const void *w_up,
                         int32_t *state, void *ws, void *stream, const Scatter *sc = nullptr) {
    int g0, S;
    int rc = expert_ffn_common(who, table, rank, T, k, d, f, dt, g0, S);
    if (rc != GRACE_OK) return rc;
    if (T == 0) return GRACE_OK;
    if (S == 0) return sc ? grace_permute_rows(sc->x, sc->pos, T, k, d, dt, (void *)xp, stream) : GRACE_OK;
    if (!xp || !inst_off || !w_gate || !w_up || !ws) return fail(GRACE_EINVAL, "%s: null device pointer", who);
    if ((((uintptr_t)xp) | ((uintptr_t)w_gate) | ((uintptr_t)w_up) | ((uintptr_t)ws)) & 15)
        return fail(GRACE_EINVAL, "%s: device pointers must be 16-byte aligned", who);
    GemmArgs up = expert_shape(true, S, d, f);
    up.A = xp; up.B0 = w_gate; up.B1 = w_up; up.out = ws;
    up.seg_off = inst_off + g0;
    up.share_state = state;
    const Rows rows = expert_rows(S, table->I, T, k);
    if (sc) {
        // the scatter rides on the projection's launch (carries_rows), or is one of its own ahead of it.  Steps, two launches -> one, us: d = 2048, k = 8, 4096 tokens of f = 1024 202 -> 187, 8000 306 -> 284, 7001 of f = 768 180 -> 172, 4000 132 -> 123; d = 4096, k = 2, f =
        // 14336, 3000 tokens 424 -> 407, 1500 and 8192 (power limit) even
        const int n_cu = compute_units();
        if (n_cu > 0 && carries_rows(route_gemm<true>(up, dt, rows, n_cu), dt, T, k, d, true)) {
            up.A = sc->src;
            up.sc_x = sc->x; up.sc_xp = (void *)xp; up.sc_pos = sc->pos; up.sc_T = T; up.sc_k = k; up.sc_row_bytes = d * 2;
            return launch_gemm<true, pers::EXPERTS_GATHER>(up, dt, rows, (hipStream_t)stream, who);
        }
        if (n_cu > 0 && joins_shared(true, T, k, d, f, 0, S, table->I, dt, n_cu)) {
            up.A = sc->src;
            up.sc_x = sc->x; up.sc_xp = (void *)xp; up.sc_pos = sc->pos; up.sc_T = T; up.sc_k = k; up.sc_row_bytes = d * 2;
            return launch_joint<true>(nullptr, rows, up, rows, n_cu, (hipStream_t)stream, who);
        }
        rc = grace_permute_rows(sc->x, sc->pos, T, k, d, dt, (void *)xp, stream);
        if (rc != GRACE_OK) return rc;
    }
    return launch_gemm<true, pers::EXPERTS>(up, dt, rows, (hipStream_t)stream, who);
}

extern "C" int grace_dispatch_ffn_up_share(const grace_table *table, int32_t local_rank, grace_policy policy, const float *logits, int32_t T,
                                           int32_t E, int32_t k, int32_t renorm, const uint32_t *rr_in, uint32_t *rr_out,
                                           int32_t *topk_expert, float *topk_weight, int32_t *topk_inst, int32_t *expert_count,
                                           const void *x, int32_t d, int32_t f, int32_t n_shared, grace_dtype dt, int32_t *perm_pos,
                                           int32_t *perm_src, int32_t *inst_off, int32_t *rank_off, int32_t *node_off, void *xp,
                                           const void *w_gate, const void *w_up, const void *shared_gate, const void *shared_up,
                                           int32_t *state, void *ws, void *ws_shared, void *stream) {
    const char *const who = "dispatch_ffn_up_share";
    if (!state) return fail(GRACE_EINVAL, "%s: state is null", who);
    if (T > 0 && !x) return fail(GRACE_EINVAL, "%s: x is null", who);
    int g0, S;
    int rc = expert_ffn_common(who, table, local_rank, T, k, d, f, dt, g0, S);
    if (rc != GRACE_OK) return rc;
    rc = check_route_args(table, local_rank, policy, logits, T, E, k, rr_in, rr_out, topk_expert, topk_weight, topk_inst, expert_count, ws);
    if (rc != GRACE_OK) return rc;
    rc = check_permute_args(table, topk_inst, T, k, x, d, dt, perm_pos, perm_src, inst_off, rank_off, node_off, xp, ws);
    if (rc == GRACE_OK && n_shared != 0) rc = shared_ffn_common(who, T, d, f, n_shared, dt);
    if (rc != GRACE_OK) return rc;
    const int n_cu = compute_units();
    if (n_cu <= 0) return fail(GRACE_EHIP, "%s: cannot query the device", who);
    auto shared_alone = [&] { return n_shared ? grace_shared_ffn_up(x, T, d, f, n_shared, dt, shared_gate, shared_up, ws_shared, stream) : GRACE_OK; };
    if (T == 0 || !joins_dispatch(table, local_rank, T, k, d, f, n_shared, dt, n_cu)) {
        rc = grace_route_permute(table, local_rank, policy, logits, T, E, k, renorm, rr_in, rr_out, topk_expert, topk_weight, topk_inst,
                                 expert_count, x, d, dt, perm_pos, perm_src, inst_off, rank_off, node_off, xp, ws, stream);
        if (rc != GRACE_OK) return rc;
        rc = expert_ffn_up(who, table, local_rank, xp, inst_off, T, k, d, f, dt, w_gate, w_up, state, ws, stream);
        return rc != GRACE_OK ? rc : shared_alone();
    }
    if (!w_gate || !w_up) return fail(GRACE_EINVAL, "%s: null device pointer", who);
    if ((((uintptr_t)w_gate) | ((uintptr_t)w_up) | ((uintptr_t)ws)) & 15) return fail(GRACE_EINVAL, "%s: device pointers must be 16-byte aligned", who);
    const GemmArgs shape = expert_shape(true, S, d, f);
    const Rows rows = expert_rows(S, table->I, T, k);
    const Route route = route_gemm<true>(shape, dt, rows, n_cu);
    const int cols = route == Route::MID ? mid::Shape<true>::BN : strm::Shape<true>::COLS;
    TinyUp a{tiny_args(table, local_rank, policy, logits, T, k, renorm, rr_in, rr_out, topk_expert, topk_weight, topk_inst, expert_count, x, d,
                       dt, perm_pos, perm_src, inst_off, rank_off, node_off, xp),
             shape, table->d_inst_span + g0, g0, policy == GRACE_POLICY_WRR, (f + cols - 1) / cols, {}, 0};
    a.up.A = x; a.up.B0 = w_gate; a.up.B1 = w_up; a.up.out = ws;
    a.up.share_state = state;
    const bool pieces = dt == GRACE_F32 && stream_pieces<4>(rows);
    // the shared experts' tiles run beside the others where they are streamed as well
    bool with_shared = false;
    if (n_shared && route == Route::STREAM && T <= strm::MAX_ROWS) {
        a.shared = shared_shape(true, T, d, f, n_shared);
        with_shared = route_gemm<true>(a.shared, dt, shared_rows(T), n_cu) == Route::STREAM;
        if (with_shared) {
            if (!shared_gate || !shared_up || !ws_shared) return fail(GRACE_EINVAL, "%s: null device pointer", who);
            if (((uintptr_t)shared_gate | (uintptr_t)shared_up | (uintptr_t)ws_shared) & 15)
                return fail(GRACE_EINVAL, "%s: device pointers must be 16-byte aligned", who);
            a.shared.A = x; a.shared.B0 = shared_gate; a.shared.B1 = shared_up; a.shared.out = ws_shared;
            a.shared_strips = (a.shared.N + cols - 1) / cols;
        }
    }
    if (route == Route::STREAM && n_shared == 0 && deals_columns(S, T, d, f, dt, n_cu)) {
        launch_tiny_cols(a, dt, n_cu, (hipStream_t)stream);
    } else if (route == Route::MID) {
        launch_tiny_up_mid(a, n_cu, (hipStream_t)stream);
    } else {
        const Grid l = dt == GRACE_BF16 ? stream_grid<true, 2>(shape, rows, n_cu, a.shared_strips) : stream_grid<true, 4>(shape, rows, n_cu, a.shared_strips);
        const int64_t tiles = (int64_t)S * a.n_strips * (pieces ? (T + strm::MAX_ROWS - 1) / strm::MAX_ROWS : 1) + a.shared_strips;
        const int waves = joined_waves(l.threads / 64, tiles, pieces, T, k, d, E, dt, n_cu);   // (stream_grid's partial sums alone may take 64 KB)
        if (tiny_up_lds(T, waves, pieces) > LDS_WITHOUT_ASKING && !allow_full_lds(tiny_up_kernel_of(dt, T, E, pieces), who)) return GRACE_EHIP;
        launch_tiny_up(a, dt, waves, pieces, n_cu, (hipStream_t)stream);
    }
    GRACE_LAUNCH_CHECK(who);
    return with_shared ? GRACE_OK : shared_alone();
}

extern "C" int grace_expert_ffn_up(const grace_table *table, int32_t rank, const void *xp, const int32_t *inst_off,
                                   int32_t T, int32_t k, int32_t d, int32_t f, grace_dtype dt, const void *w_gate,
                                   const void *w_up, void *ws, void *stream) {
    return expert_ffn_up("expert_ffn_up", table, rank, xp, inst_off, T, k, d, f, dt, w_gate, w_up, nullptr, ws, stream);
}

extern "C" int grace_expert_ffn_up_share(const grace_table *table, int32_t rank, const void *xp, const int32_t *inst_off,
                                         int32_t T, int32_t k, int32_t d, int32_t f, grace_dtype dt, const void *w_gate,
                                         const void *w_up, int32_t *state, void *ws, void *stream) {
    if (!state) return fail(GRACE_EINVAL, "expert_ffn_up_share: state is null");
    return expert_ffn_up("expert_ffn_up_share", table, rank, xp, inst_off, T, k, d, f, dt, w_gate, w_up, state, ws, stream);
}

extern "C" int grace_expert_ffn_up_share_scatter(const grace_table *table, int32_t rank, const void *x, const int32_t *perm_pos,
                                                 const int32_t *perm_src, void *xp, const int32_t *inst_off, int32_t T, int32_t k,
                                                 int32_t d, int32_t f, grace_dtype dt, const void *w_gate, const void *w_up,
                                                 int32_t *state, void *ws, void *stream) {
    if (!state) return fail(GRACE_EINVAL, "expert_ffn_up_share_scatter: state is null");
    if (T > 0 && (!x || !perm_pos || !perm_src || !xp)) return fail(GRACE_EINVAL, "expert_ffn_up_share_scatter: null device pointer");
    if (((uintptr_t)x | (uintptr_t)xp) & 15) return fail(GRACE_EINVAL, "expert_ffn_up_share_scatter: x and xp must be 16-byte aligned");
    const Scatter sc = {x, perm_pos, perm_src};
    return expert_ffn_up("expert_ffn_up_share_scatter", table, rank, xp, inst_off, T, k, d, f, dt, w_gate, w_up, state, ws, stream, &sc);
}

static_assert(SHARE_STATE_INTS == GRACE_SHARE_STATE_INTS, "header and kernels must agree on the state size");

static int expert_ffn_down(const char *who, const grace_table *table, int32_t rank, const int32_t *inst_off, int32_t T,
                           int32_t k, int32_t d, int32_t f, grace_dtype dt, const void *w_down, void *y, int32_t *state,
                           bool clear_others, void *ws, void *stream, int joined_shared = -1 /* of a joined step: shared experts */) {
    int g0, S;
    int rc = expert_ffn_common(who, table, rank, T, k, d, f, dt, g0, S);
    if (rc != GRACE_OK) return rc;
    if (T == 0 || (S == 0 && !clear_others)) return GRACE_OK;
    if (!y || (S > 0 && (!inst_off || !w_down || !ws))) return fail(GRACE_EINVAL, "%s: null device pointer", who);
    if ((((uintptr_t)w_down) | ((uintptr_t)y) | ((uintptr_t)ws)) & 15)
        return fail(GRACE_EINVAL, "%s: device pointers must be 16-byte aligned", who);
    const size_t el = dt == GRACE_F32 ? 4 : 2;
    if ((state || clear_others) && ((size_t)d * el) % 16 != 0)
        return fail(GRACE_ESHAPE, "%s: row of %zu bytes is not a multiple of 16", who, (size_t)d * el);
    if (S == 0) {   // every row is another rank's
        const int64_t n = (int64_t)T * k * (int64_t)((size_t)d * el / 16);
        zero_fill_kernel<<<(unsigned)std::min<int64_t>((n + 255) / 256, 4096), 256, 0, (hipStream_t)stream>>>((uint4 *)y, n);
        GRACE_LAUNCH_CHECK(who);
        return GRACE_OK;
    }
    GemmArgs dn = expert_shape(false, S, d, f);
    dn.A = ws; dn.B0 = w_down; dn.out = y;
    dn.seg_off = inst_off + g0;
    if (joined_shared >= 0) {
        const int n_cu = compute_units();
        if (n_cu <= 0) return fail(GRACE_EHIP, "%s: cannot query the device", who);
        if (joins_dispatch(table, rank, T, k, d, f, joined_shared, dt, n_cu)) dn.a_slot_rows = T;
    }
    dn.share_state = state; dn.stale = state ? 1 : clear_others ? 2 : 0; dn.share_rows = (int64_t)T * k; dn.share_row_vec = (int)((size_t)d * el / 16);
    return launch_gemm<false, pers::EXPERTS>(dn, dt, expert_rows(S, table->I, T, k), (hipStream_t)stream, who);
}

extern "C" int grace_expert_ffn_down(const grace_table *table, int32_t rank, const int32_t *inst_off, int32_t T,
                                     int32_t k, int32_t d, int32_t f, grace_dtype dt, const void *w_down, void *y,
                                     void *ws, void *stream) {
    return expert_ffn_down("expert_ffn_down", table, rank, inst_off, T, k, d, f, dt, w_down, y, nullptr, false, ws, stream);
}

extern "C" int grace_expert_ffn_down_fresh(const grace_table *table, int32_t rank, const int32_t *inst_off, int32_t T,
                                           int32_t k, int32_t d, int32_t f, grace_dtype dt, const void *w_down, void *y,
                                           void *ws, void *stream) {
    return expert_ffn_down("expert_ffn_down_fresh", table, rank, inst_off, T, k, d, f, dt, w_down, y, nullptr, true, ws, stream);
}

extern "C" int grace_expert_ffn_down_share(const grace_table *table, int32_t rank, const int32_t *inst_off, int32_t T,
                                           int32_t k, int32_t d, int32_t f, grace_dtype dt, const void *w_down, void *y,
                                           int32_t *state, void *ws, void *stream) {
    if (!state) return fail(GRACE_EINVAL, "expert_ffn_down_share: state is null");
    return expert_ffn_down("expert_ffn_down_share", table, rank, inst_off, T, k, d, f, dt, w_down, y, state, false, ws, stream);
}

extern "C" int grace_dispatch_ffn_down_share(const grace_table *table, int32_t rank, const int32_t *inst_off, const int32_t *perm_pos,
                                             const float *topk_weight, int32_t T, int32_t k, int32_t d, int32_t f, int32_t n_shared,
                                             grace_dtype dt, const void *w_down, const void *shared_down, void *y, void *y_shared,
                                             int32_t *state, void *ws, void *ws_shared, void *out, void *stream) {
    const char *const who = "dispatch_ffn_down_share";
    if (!state) return fail(GRACE_EINVAL, "%s: state is null", who);
    int g0, S;
    int rc = expert_ffn_common(who, table, rank, T, k, d, f, dt, g0, S);
    if (rc == GRACE_OK && n_shared != 0) rc = shared_ffn_common(who, T, d, f, n_shared, dt);
    if (rc != GRACE_OK) return rc;
    const int n_cu = compute_units();
    if (n_cu <= 0) return fail(GRACE_EHIP, "%s: cannot query the device", who);
    if (T == 0 || !out || !joins_dispatch(table, rank, T, k, d, f, n_shared, dt, n_cu) || !joins_combine(T, k, d, f, n_shared, S, dt, n_cu)) {
        rc = expert_ffn_down(who, table, rank, inst_off, T, k, d, f, dt, w_down, y, state, false, ws, stream, n_shared);
        if (rc == GRACE_OK && n_shared) rc = grace_shared_ffn_down(T, d, f, n_shared, dt, shared_down, y_shared, ws_shared, stream);
        if (rc != GRACE_OK || !out) return rc;
        const void *ys = n_shared ? y_shared : nullptr;
        return S == table->I ? grace_combine(y, perm_pos, topk_weight, T, k, d, dt, ys, out, stream)
                             : grace_combine_share(y, perm_pos, topk_weight, T, k, d, dt, ys, state, out, stream);
    }
    if (!inst_off || !perm_pos || !topk_weight || !w_down || !y || !ws || (n_shared && (!shared_down || !y_shared || !ws_shared)))
        return fail(GRACE_EINVAL, "%s: null device pointer", who);
    uintptr_t at = (uintptr_t)w_down | (uintptr_t)y | (uintptr_t)ws | (uintptr_t)out;
    if (n_shared) at |= (uintptr_t)shared_down | (uintptr_t)y_shared | (uintptr_t)ws_shared;
    if (at & 15) return fail(GRACE_EINVAL, "%s: device pointers must be 16-byte aligned", who);
    TinyDown a{};
    a.experts = expert_shape(false, S, d, f);
    a.experts.A = ws; a.experts.B0 = w_down; a.experts.out = y;
    a.experts.seg_off = inst_off + g0;
    a.experts.a_slot_rows = T;
    a.experts.share_state = state; a.experts.stale = 1; a.experts.share_rows = (int64_t)T * k; a.experts.share_row_vec = (int)((size_t)d * (dt == GRACE_F32 ? 4 : 2) / 16);
    if (n_shared) {
        a.shared = shared_shape(false, T, d, f, n_shared);
        a.shared.A = ws_shared; a.shared.B0 = shared_down; a.shared.out = y_shared;
    }
    a.perm_pos = perm_pos; a.weight = topk_weight; a.out = out;
    a.T = T; a.k = k; a.n_shared = n_shared;
    if (!allow_full_lds(tiny_down_kernel_of(dt, T, d, n_cu), who)) return GRACE_EHIP;
    launch_tiny_down(a, dt, tiny_down_lds(T, k, S, n_shared, d, n_cu), n_cu, (hipStream_t)stream);
    GRACE_LAUNCH_CHECK(who);
    return GRACE_OK;
}

extern "C" int grace_dispatch_joins_ffn(const grace_table *table, int32_t local_rank, int32_t T, int32_t k, int32_t d, int32_t f,
                                        int32_t n_shared, grace_dtype dt, int32_t n_cu, int32_t *joined) {
    if (!joined) return fail(GRACE_EINVAL, "dispatch_joins_ffn: null output");
    int g0, S;
    int rc = expert_ffn_common("dispatch_joins_ffn", table, local_rank, T, k, d, f, dt, g0, S);
    if (rc == GRACE_OK && n_shared != 0) rc = shared_ffn_common("dispatch_joins_ffn", T, d, f, n_shared, dt);
    if (rc != GRACE_OK) return rc;
    if (n_cu == 0) n_cu = compute_units();
    if (n_cu <= 0) return fail(GRACE_EHIP, "dispatch_joins_ffn: cannot query the device");
    *joined = T == 0 || !joins_dispatch(table, local_rank, T, k, d, f, n_shared, dt, n_cu) ? 0 : joins_combine(T, k, d, f, n_shared, S, dt, n_cu) ? 2 : 1;
    return GRACE_OK;
}

extern "C" int grace_expert_ffn(const grace_table *table, int32_t rank, const void *xp, const int32_t *inst_off,
                                int32_t T, int32_t k, int32_t d, int32_t f, grace_dtype dt, const void *w_gate,
                                const void *w_up, const void *w_down, void *y, void *ws, void *stream) {
    int rc = grace_expert_ffn_up(table, rank, xp, inst_off, T, k, d, f, dt, w_gate, w_up, ws, stream);
    if (rc != GRACE_OK) return rc;
    return grace_expert_ffn_down(table, rank, inst_off, T, k, d, f, dt, w_down, y, ws, stream);
}

static int shared_ffn_common(const char *who, int32_t T, int32_t d, int32_t f, int32_t n_shared, grace_dtype dt) {
    if (T < 0 || n_shared < 1) return fail(GRACE_EINVAL, "%s: T=%d, n_shared=%d invalid", who, T, n_shared);
    int rc = check_ffn_shapes(who, d, f, dt);
    if (rc != GRACE_OK) return rc;
    if ((int64_t)n_shared * f > INT32_MAX) return fail(GRACE_ESHAPE, "%s: n_shared*f too large", who);
    return GRACE_OK;
}

static int shared_ffn_up(const char *who, const void *x, int32_t T, int32_t d, int32_t f, int32_t n_shared, grace_dtype dt,
                         const void *w_gate, const void *w_up, void *ws, const int32_t *perm_pos, int32_t k, void *xp,
                         void *stream) {
    int rc = shared_ffn_common(who, T, d, f, n_shared, dt);
    if (rc != GRACE_OK) return rc;
    if (T == 0) return GRACE_OK;
    if (!x || !w_gate || !w_up || !ws) return fail(GRACE_EINVAL, "%s: null device pointer", who);
    if ((((uintptr_t)x) | ((uintptr_t)w_gate) | ((uintptr_t)w_up) | ((uintptr_t)ws)) & 15)
        return fail(GRACE_EINVAL, "%s: device pointers must be 16-byte aligned", who);
    GemmArgs up = shared_shape(true, T, d, f, n_shared);
    up.A = x; up.B0 = w_gate; up.B1 = w_up; up.out = ws;
    if (perm_pos) {
        // the row scatter rides on the projection's launch, or is one of its own ahead of it
        const int n_cu = compute_units();
        if (n_cu > 0 && carries_rows(route_gemm<true>(up, dt, shared_rows(T), n_cu), dt, T, k, d, false)) {
            up.sc_x = x; up.sc_xp = xp; up.sc_pos = perm_pos; up.sc_T = T; up.sc_k = k; up.sc_row_bytes = d * 2;
        } else {
            rc = grace_permute_rows(x, perm_pos, T, k, d, dt, xp, stream);
            if (rc != GRACE_OK) return rc;
        }
    }
    return launch_gemm<true, pers::SHARED>(up, dt, shared_rows(T), (hipStream_t)stream, who);
}

extern "C" int grace_shared_ffn_up(const void *x, int32_t T, int32_t d, int32_t f, int32_t n_shared, grace_dtype dt,
                                   const void *w_gate, const void *w_up, void *ws, void *stream) {
    return shared_ffn_up("shared_ffn_up", x, T, d, f, n_shared, dt, w_gate, w_up, ws, nullptr, 0, nullptr, stream);
}

extern "C" int grace_shared_ffn_up_scatter(const void *x, int32_t T, int32_t d, int32_t f, int32_t n_shared, grace_dtype dt,
                                           const void *w_gate, const void *w_up, void *ws, const int32_t *perm_pos,
                                           int32_t k, void *xp, void *stream) {
    if (k < 1) return fail(GRACE_EINVAL, "shared_ffn_up_scatter: k=%d invalid", k);
    if (T > 0 && (!perm_pos || !xp)) return fail(GRACE_EINVAL, "shared_ffn_up_scatter: null device pointer");
    if (((uintptr_t)xp) & 15) return fail(GRACE_EINVAL, "shared_ffn_up_scatter: xp must be 16-byte aligned");
    if ((int64_t)T * k > INT32_MAX) return fail(GRACE_ESHAPE, "shared_ffn_up_scatter: T*k exceeds 2^31-1");
    return shared_ffn_up("shared_ffn_up_scatter", x, T, d, f, n_shared, dt, w_gate, w_up, ws, perm_pos, k, xp, stream);
}

extern "C" int grace_shared_ffn_down(int32_t T, int32_t d, int32_t f, int32_t n_shared, grace_dtype dt,
                                     const void *w_down, void *y_shared, void *ws, void *stream) {
    int rc = shared_ffn_common("shared_ffn_down", T, d, f, n_shared, dt);
    if (rc != GRACE_OK) return rc;
    if (T == 0) return GRACE_OK;
    if (!w_down || !y_shared || !ws) return fail(GRACE_EINVAL, "shared_ffn_down: null device pointer");
    if ((((uintptr_t)w_down) | ((uintptr_t)y_shared) | ((uintptr_t)ws)) & 15)
        return fail(GRACE_EINVAL, "shared_ffn_down: device pointers must be 16-byte aligned");
    GemmArgs dn = shared_shape(false, T, d, f, n_shared);
    dn.A = ws; dn.B0 = w_down; dn.out = y_shared;
    return launch_gemm<false, pers::SHARED>(dn, dt, shared_rows(T), (hipStream_t)stream, "shared_ffn down projection");
}

extern "C" int grace_shared_ffn(const void *x, int32_t T, int32_t d, int32_t f, int32_t n_shared, grace_dtype dt,
                                const void *w_gate, const void *w_up, const void *w_down, void *y_shared, void *ws,
                                void *stream) {
    int rc = shared_ffn_common("shared_ffn", T, d, f, n_shared, dt);
    if (rc != GRACE_OK) return rc;
    if (T == 0) return GRACE_OK;
    if (!w_down || !y_shared) return fail(GRACE_EINVAL, "shared_ffn: null device pointer");
    rc = grace_shared_ffn_up(x, T, d, f, n_shared, dt, w_gate, w_up, ws, stream);
    if (rc != GRACE_OK) return rc;
    return grace_shared_ffn_down(T, d, f, n_shared, dt, w_down, y_shared, ws, stream);
}

extern "C" int grace_expert_shared_ffn_up_scatter(const grace_table *table, int32_t rank, const void *x, const int32_t *perm_pos,
                                                  const int32_t *perm_src, void *xp, const int32_t *inst_off, int32_t T, int32_t k,
                                                  int32_t d, int32_t f, int32_t n_shared, grace_dtype dt, const void *w_gate,
                                                  const void *w_up, const void *shared_gate, const void *shared_up, int32_t *state,
                                                  void *ws, void *ws_shared, void *stream) {
    const char *const who = "expert_shared_ffn_up_scatter";
    int g0, S;
    int rc = expert_ffn_common(who, table, rank, T, k, d, f, dt, g0, S);
    if (rc == GRACE_OK) rc = shared_ffn_common(who, T, d, f, n_shared, dt);
    if (rc != GRACE_OK) return rc;
    if (!state) return fail(GRACE_EINVAL, "%s: state is null", who);
    const int n_cu = compute_units();
    if (n_cu <= 0 || !joins_shared(true, T, k, d, f, n_shared, S, table->I, dt, n_cu)) {
        rc = grace_shared_ffn_up_scatter(x, T, d, f, n_shared, dt, shared_gate, shared_up, ws_shared, perm_pos, k, xp, stream);
        return rc != GRACE_OK ? rc : grace_expert_ffn_up_share(table, rank, xp, inst_off, T, k, d, f, dt, w_gate, w_up, state, ws, stream);
    }
    if (!x || !perm_pos || !perm_src || !xp || !inst_off || !w_gate || !w_up || !shared_gate || !shared_up || !ws || !ws_shared)
        return fail(GRACE_EINVAL, "%s: null device pointer", who);
    if (((uintptr_t)x | (uintptr_t)xp | (uintptr_t)w_gate | (uintptr_t)w_up | (uintptr_t)shared_gate | (uintptr_t)shared_up | (uintptr_t)ws |
         (uintptr_t)ws_shared) & 15)
        return fail(GRACE_EINVAL, "%s: device pointers must be 16-byte aligned", who);
    GemmArgs all = shared_shape(true, T, d, f, n_shared), up = expert_shape(true, S, d, f);
    all.A = x; all.B0 = shared_gate; all.B1 = shared_up; all.out = ws_shared;
    up.A = perm_src; up.B0 = w_gate; up.B1 = w_up; up.out = ws;
    up.seg_off = inst_off + g0;
    up.share_state = state;
    up.sc_x = x; up.sc_xp = xp; up.sc_pos = perm_pos; up.sc_T = T; up.sc_k = k; up.sc_row_bytes = d * 2;
    return launch_joint<true>(&all, shared_rows(T), up, expert_rows(S, table->I, T, k), n_cu, (hipStream_t)stream, who);
}

extern "C" int grace_expert_shared_ffn_down(const grace_table *table, int32_t rank, const int32_t *inst_off, int32_t T, int32_t k, int32_t d,
                                            int32_t f, int32_t n_shared, grace_dtype dt, const void *w_down, const void *shared_down,
                                            void *y, void *y_shared, int32_t *state, void *ws, void *ws_shared, void *stream) {
    const char *const who = "expert_shared_ffn_down";
    int g0, S;
    int rc = expert_ffn_common(who, table, rank, T, k, d, f, dt, g0, S);
    if (rc == GRACE_OK) rc = shared_ffn_common(who, T, d, f, n_shared, dt);
    if (rc != GRACE_OK) return rc;
    if (!state) return fail(GRACE_EINVAL, "%s: state is null", who);
    const int n_cu = compute_units();
    if (n_cu <= 0 || !joins_shared(false, T, k, d, f, n_shared, S, table->I, dt, n_cu)) {
        rc = grace_expert_ffn_down_share(table, rank, inst_off, T, k, d, f, dt, w_down, y, state, ws, stream);
        return rc != GRACE_OK ? rc : grace_shared_ffn_down(T, d, f, n_shared, dt, shared_down, y_shared, ws_shared, stream);
    }
    if (!inst_off || !w_down || !shared_down || !y || !y_shared || !ws || !ws_shared) return fail(GRACE_EINVAL, "%s: null device pointer", who);
    if (((uintptr_t)w_down | (uintptr_t)shared_down | (uintptr_t)y | (uintptr_t)y_shared | (uintptr_t)ws | (uintptr_t)ws_shared) & 15)
        return fail(GRACE_EINVAL, "%s: device pointers must be 16-byte aligned", who);
    GemmArgs all = shared_shape(false, T, d, f, n_shared), dn = expert_shape(false, S, d, f);
    all.A = ws_shared; all.B0 = shared_down; all.out = y_shared;
    dn.A = ws; dn.B0 = w_down; dn.out = y;
    dn.seg_off = inst_off + g0;
    dn.share_state = state; dn.stale = 1; dn.share_rows = (int64_t)T * k; dn.share_row_vec = d * 2 / 16;
    return launch_joint<false>(&all, shared_rows(T), dn, expert_rows(S, table->I, T, k), n_cu, (hipStream_t)stream, who);
}

extern "C" int grace_ffn_joins_shared(int32_t up, int32_t T, int32_t k, int32_t d, int32_t f, int32_t n_shared, int32_t S, int32_t I, grace_dtype dt,
                                      int32_t n_cu, int32_t *joined) {
    if (!joined) return fail(GRACE_EINVAL, "ffn_joins_shared: null output");
    if (T < 1 || k < 1 || n_shared < 0 || S < 0 || I < S || n_cu < 0)
        return fail(GRACE_EINVAL, "ffn_joins_shared: T=%d, k=%d, n_shared=%d, S=%d, I=%d, n_cu=%d invalid", T, k, n_shared, S, I, n_cu);
    const int rc = shared_ffn_common("ffn_joins_shared", T, d, f, std::max(n_shared, 1), dt);
    if (rc != GRACE_OK) return rc;
    if ((int64_t)T * k > INT32_MAX) return fail(GRACE_ESHAPE, "ffn_joins_shared: T*k exceeds 2^31-1");
    if (n_cu == 0) n_cu = compute_units();
    if (n_cu <= 0) return fail(GRACE_EHIP, "ffn_joins_shared: cannot query the device");
    *joined = joins_shared(up, T, k, d, f, n_shared, S, I, dt, n_cu);
    return GRACE_OK;
}

extern "C" int grace_ffn_kernel(int32_t up, int32_t T, int32_t k, int32_t d, int32_t f, int32_t n_shared, int32_t S, int32_t I,
                                grace_dtype dt, int32_t n_cu, int32_t *kernel, int64_t *work_items) {
    if (!kernel || !work_items) return fail(GRACE_EINVAL, "ffn_kernel: null output");
    if (T < 1 || k < 1 || n_shared < 0 || n_cu < 0) return fail(GRACE_EINVAL, "ffn_kernel: T=%d, k=%d, n_shared=%d, n_cu=%d invalid", T, k, n_shared, n_cu);
    if (n_shared == 0 && (S < 1 || I < S)) return fail(GRACE_EINVAL, "ffn_kernel: S=%d, I=%d invalid", S, I);
    int rc = n_shared > 0 ? shared_ffn_common("ffn_kernel", T, d, f, n_shared, dt) : check_ffn_shapes("ffn_kernel", d, f, dt);
    if (rc != GRACE_OK) return rc;
    if (n_shared == 0 && (int64_t)T * k > INT32_MAX) return fail(GRACE_ESHAPE, "ffn_kernel: T*k exceeds 2^31-1");
    if (n_cu == 0) n_cu = compute_units();
    if (n_cu <= 0) return fail(GRACE_EHIP, "ffn_kernel: cannot query the device");
    const GemmArgs g = n_shared > 0 ? shared_shape(up, T, d, f, n_shared) : expert_shape(up, S, d, f);
    const Rows rows = n_shared > 0 ? shared_rows(T) : expert_rows(S, I, T, k);
    const Route r = up ? route_gemm<true>(g, dt, rows, n_cu) : route_gemm<false>(g, dt, rows, n_cu);
    const Grid l = up ? grid_of<true>(r, g, dt, rows, n_cu) : grid_of<false>(r, g, dt, rows, n_cu);
    *kernel = (int32_t)r;
    *work_items = l.groups * l.threads;
    return GRACE_OK;
}

extern "C" int grace_ffn_carries_rows(int32_t T, int32_t k, int32_t d, int32_t f, int32_t n_shared, int32_t S, int32_t I, grace_dtype dt,
                                      int32_t n_cu, int32_t *carried) {
    if (!carried) return fail(GRACE_EINVAL, "ffn_carries_rows: null output");
    int32_t kernel;
    int64_t work_items;
    const int rc = grace_ffn_kernel(1, T, k, d, f, n_shared, S, I, dt, n_cu, &kernel, &work_items);
    if (rc == GRACE_OK) *carried = carries_rows((Route)kernel, dt, T, k, d, n_shared == 0);
    return rc;
}
