// The experts' gate+up projection of the smallest batches without waiting for the dispatch.
//
// The projection of a few tokens needs little of the dispatch: which tokens chose the expert of its slot.  An expert is among a
// token's k choices if fewer than k experts are ahead of it, which is one comparison with the token's logits and a count of
// bits, so every workgroup finds the rows of its slot by itself, from the logits, and reads them from the tokens.  The
// dispatch, whose results only later launches and the caller need, runs beside it in T workgroups of the same launch
// (tiny_dispatch).  As the offsets are not known yet, a slot's rows of the hidden activation begin at slot * T.
//
// Bound by latency and then by the weights, as gemm_stream_kernel; what is saved is most of the dispatch's launch (the rows cost 1.5 to 2 us, mainly the
// wait for the logits).  Dispatch and projection, two launches -> one: 1 token, 64 experts, k = 8 6.1 + 7.8 -> 9.3 us, 16 of 128 experts 9.4 + 12.1
// -> 15.0 (the first is ffn_tiny_cols.hip's now), 256 of 8, k = 2, fp32 10.3 + 6.5 -> 9.6.  Layer steps of 1 to 64 tokens (158 of five shapes, whole and a quarter of the expert
// width, both policies, replayed from a graph) take 1.02 to 1.42 times as long with two, in the median 1.16.  Where more workgroups than are resident at a time
// repeat the search for rows, many of them for tiles with work, it is even (fp32, d = 1024, f = 2816, 64 tokens 90.8 -> 91.7 us), and so are pieces of 64
// rows past two workgroups per compute unit slower (f = 704, 80 tokens 40.5 -> 50.8): the two launches there (joins_dispatch).
#include <type_traits>

#include "ffn_tiny.h"
#include "gemm_stream.h"

namespace grace {

template <int VPL, Gate GATE, int EL, int MF, bool PIECES>
__global__ __launch_bounds__(64 * strm::MAX_WAVES) void tiny_up_kernel(const TinyUp a) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int T = a.dispatch.T;
    if ((int)blockIdx.x < T) {
        TinyLds &s = *(TinyLds *)smem;
        tiny_dispatch<VPL, GATE, GATE == Gate::ROWS ? 2 : GATE == Gate::LANES ? 1 : VPL == 1 ? 1 : 4, false>(a.dispatch, (int)blockIdx.x, s);
        tiny_share_record(a, s);
        return;
    }
    if (!PIECES) {
        const int strip = (int)blockIdx.x - T - a.up.S * a.n_strips;
        if (strip >= 0)
            return strm::rows_any<true, EL, MF>(a.shared, 0, {0, T, 0, nullptr}, strip * strm::Shape<true>::COLS, (float4 *)smem);
    }
    TinyRows &s = *(TinyRows *)smem;
    const int pieces = PIECES ? (T + a.piece_rows - 1) / a.piece_rows : 1, b = (int)blockIdx.x - T;
    int slot, strip, piece = 0;
    if (PIECES) {   // pieces of the same weights next to each other on one XCD, and hot and cold slots on every one
        const int total = a.up.S * a.n_strips * pieces, each = (total + 7) >> 3, j = b >> 3, t = (b & 7) * each + j;
        if (j >= each || t >= total) return;
        strip = t / (a.up.S * pieces);
        slot = t / pieces - strip * a.up.S;
        piece = t % pieces;
    } else {
        slot = b / a.n_strips;
        strip = b - slot * a.n_strips;
    }
    const int n = rows_of_slot<VPL>(a, slot, s);
    int first = 0, end = n;
    if (PIECES && n > 0) {
        const int parts = (n + a.piece_rows - 1) / a.piece_rows, rows = ((n + parts - 1) / parts + 15) & ~15;
        first = piece * rows;
        end = min(n, first + rows);
    }
    if (first < end)
        strm::rows_any<true, EL, MF, true>(a.up, slot, {slot * T + first, slot * T + end, 0, s.list + first}, strip * strm::Shape<true>::COLS,
                                           (float4 *)(smem + ROWS_BYTES));
}

static int up_fragments(int T, bool pieces) { return pieces ? 4 : T <= 16 ? 1 : T <= 32 ? 2 : 4; }
int tiny_up_lds(int T, int waves, bool pieces) { return std::max((int)sizeof(TinyLds), ROWS_BYTES + strm::lds_bytes(waves, up_fragments(T, pieces))); }

const void *tiny_up_kernel_of(grace_dtype dt, int T, int E, bool pieces) {
    const int mf = up_fragments(T, pieces);
    auto by_rows = [&](auto vpl, auto gate, auto el) {
        constexpr int VPL = decltype(vpl)::value, EL = decltype(el)::value;
        constexpr Gate GATE = decltype(gate)::value;
        if constexpr (EL == 4 && VPL == 1 && GATE != Gate::WAVE) {
            if (pieces) return (const void *)tiny_up_kernel<VPL, GATE, EL, 4, true>;
        }
        if constexpr (!(VPL == 1 && GATE == Gate::WAVE)) {
            if (mf == 2) return (const void *)tiny_up_kernel<VPL, GATE, EL, 2, false>;
            if constexpr (VPL == 1) {
                if (mf == 4) return (const void *)tiny_up_kernel<VPL, GATE, EL, 4, false>;
            }
        }
        return (const void *)tiny_up_kernel<VPL, GATE, EL, 1, false>;
    };
    auto by_gate = [&](auto el) {
        using std::integral_constant;
        if (E > 128) return by_rows(integral_constant<int, 4>{}, integral_constant<Gate, Gate::WAVE>{}, el);
        if (E > 64) return by_rows(integral_constant<int, 2>{}, integral_constant<Gate, Gate::WAVE>{}, el);
        if (T <= 4) return by_rows(integral_constant<int, 1>{}, integral_constant<Gate, Gate::WAVE>{}, el);
        if (E <= TINY_LANE_E) return by_rows(integral_constant<int, 1>{}, integral_constant<Gate, Gate::LANES>{}, el);
        return by_rows(integral_constant<int, 1>{}, integral_constant<Gate, Gate::ROWS>{}, el);
    };
    return dt == GRACE_BF16 ? by_gate(std::integral_constant<int, 2>{}) : by_gate(std::integral_constant<int, 4>{});
}

void launch_tiny_up(const TinyUp &tiles, grace_dtype dt, int waves, bool pieces, int n_cu, hipStream_t st) {
    TinyUp a = tiles;
    const int T = a.dispatch.T;
    a.piece_rows = strm::MAX_ROWS;
    auto tiles_of = [&] { return a.up.S * a.n_strips * ((T + a.piece_rows - 1) / a.piece_rows); };
    while (pieces && a.piece_rows > 16 && 2 * tiles_of() <= n_cu) a.piece_rows /= 2;   // as gemm_stream_tiles_kernel's, of the tiles that there may be
    const int blocks = pieces ? (tiles_of() + 7) / 8 * 8 : a.up.S * a.n_strips + a.shared_strips;
    void *params[] = {&a};
    (void)hipLaunchKernel(tiny_up_kernel_of(dt, T, a.dispatch.E, pieces), dim3((unsigned)(T + blocks)), dim3(waves * 64), params, tiny_up_lds(T, waves, pieces), st);
}

}  // namespace grace
