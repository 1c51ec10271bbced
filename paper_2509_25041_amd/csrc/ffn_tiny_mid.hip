// ffn_tiny.hip's launch where the 96-row kernel takes the projection: more than 16 tokens and tiles enough to fill the chip.
//
// Which slots have rows, and so how many tiles there are, would take the whole gate of every workgroup (64 tokens, k = 8, 64 experts: 30.3 us
// with that, 26.5 without; dispatch and projection by themselves 9.4 + 22.4), so tiles are numbered as if all slots had rows, one piece
// each, and workgroups of a slot without rows leave.  With more of these tiles than compute units, some of which then get two that work while others
// have none, the joined launch is no faster (steps of 24 to 96 tokens, 288 tiles 0.94 to 1.02): the two launches then.  Layer
// steps, two launches -> one: d = 2048, f = 1024, 16 slots, 64 tokens 53.7 -> 47.8 us, 17 36.4 -> 34.1; f = 1408, 7 slots, 80 tokens 91.8 -> 91.9 (k = 4);
// d = 4096, f = 3584, one slot, 96 tokens 48.2 -> 42.3.
#include <type_traits>

#include "ffn_tiny.h"
#include "gemm_bf16_mid.h"

namespace grace {

static_assert(sizeof(TinyLds) <= mid::LDS_BYTES, "the dispatch works in the tiles' LDS");
static_assert(mid::BM <= mid::THREADS, "a thread per token");

// (as gemm_bf16_mid_kernel)
__host__ __device__ inline bool tiny_halves(int total, int K, int n_cu) { return K >= 4 * mid::BK && 2 * total <= n_cu; }

template <int VPL, Gate GATE>
__global__ __launch_bounds__(mid::THREADS, 2) void tiny_up_mid_kernel(const TinyUp a, int n_cu) {
    __shared__ __attribute__((aligned(1024))) char smem[mid::LDS_BYTES];
    __shared__ TinyRows s;
    const int T = a.dispatch.T;
    if ((int)blockIdx.x < T) {
        tiny_dispatch<VPL, GATE, GATE == Gate::LANES ? 1 : VPL == 1 ? 6 : 2, false>(a.dispatch, (int)blockIdx.x, *(TinyLds *)smem);
        tiny_share_record(a, *(const TinyLds *)smem);
        return;
    }
    const int total = a.up.S * a.n_strips;
    const bool halves = tiny_halves(total, a.up.K, n_cu);
    const int number = mid::of_runs((int)blockIdx.x - T, halves ? 2 * total : total);
    if (number < 0) return;
    const int t = halves ? number >> 1 : number, slot = t / a.n_strips, strip = t - slot * a.n_strips;
    const int n0 = strip * mid::Shape<true>::BN + (halves ? (number & 1) * (mid::Shape<true>::BN / 2) : 0);
    if (n0 >= a.up.N) return;
    const int n = rows_of_slot<VPL>(a, slot, s);
    const int m0 = slot * T, m_end = m0 + n, first_step = t / 4 % ((a.up.K + mid::BK - 1) / mid::BK);
    auto tile = [&](auto nj) {
        constexpr int NJ = decltype(nj)::value;
        if (n > 64) mid::tile_body<true, false, 6, NJ, mid::RowsFrom::LIST>(a.up, slot, m0, m_end, 0, n0, first_step, smem, s.list);
        else if (n > 32) mid::tile_body<true, false, 4, NJ, mid::RowsFrom::LIST>(a.up, slot, m0, m_end, 0, n0, first_step, smem, s.list);
        else if (n > 0) mid::tile_body<true, false, 2, NJ, mid::RowsFrom::LIST>(a.up, slot, m0, m_end, 0, n0, first_step, smem, s.list);
    };
    if (halves) tile(std::integral_constant<int, 1>{});
    else tile(std::integral_constant<int, 2>{});
}

int64_t tiny_up_mid_blocks(int S, int K, int n_strips, int n_cu) {
    const int64_t total = (int64_t)S * n_strips;
    return total > n_cu ? 0 : (total * (tiny_halves((int)total, K, n_cu) ? 2 : 1) + 63) / 64 * 64;
}

void launch_tiny_up_mid(const TinyUp &a, int n_cu, hipStream_t st) {
    const int T = a.dispatch.T, E = a.dispatch.E;
    const int64_t blocks = tiny_up_mid_blocks(a.up.S, a.up.K, a.n_strips, n_cu);
    auto *kernel = E <= TINY_LANE_E ? tiny_up_mid_kernel<1, Gate::LANES> : E <= 64 ? tiny_up_mid_kernel<1, Gate::ROWS>
                   : E <= 128 ? tiny_up_mid_kernel<2, Gate::ROWS> : tiny_up_mid_kernel<4, Gate::WAVE>;
    kernel<<<(unsigned)(T + blocks), mid::THREADS, 0, st>>>(a, n_cu);
}

}  // namespace grace
