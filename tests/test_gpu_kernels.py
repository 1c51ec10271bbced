"""Kernel variants that the launchers choose by size, each at the sizes where it can go wrong, against the
oracle: edges of its tiles, remainders along every axis, both ends of its range."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

import oracle
import paper_2509_25041_amd as grace
import test_gpu_parity as parity
from test_gpu_parity import TOL, host, rel_err
from workloads import LayerConfig, make_workload

pytestmark = pytest.mark.gpu


def ffn_of_segments(seg_rows, T, k, d, f, dtype=torch.bfloat16, seed=0):
    """Expert FFN of one rank that hosts every expert, on given row segments of a [T * k, d] buffer, and the
    oracle's rows."""
    E = len(seg_rows)
    rng = np.random.default_rng(seed)

    def normal(scale, *shape):
        return torch.from_numpy((scale * rng.standard_normal(shape)).astype(np.float32)).cuda().to(dtype)

    table = grace.GraceTable(E, 1, 1, [0], [1], list(range(E + 1)), [0] * E)
    xp = normal(1.0, T * k, d)
    wg, wu, wd = normal(0.05, E, f, d), normal(0.05, E, f, d), normal(0.05, E, d, f)
    off = np.concatenate([[0], np.cumsum(seg_rows)]).astype(np.int32)
    y = torch.full((T * k, d), 7.0, dtype=dtype, device="cuda")
    grace.grace_expert_ffn(table, 0, xp, torch.from_numpy(off).cuda(), T, k, wg, wu, wd, y=y)
    torch.cuda.synchronize()
    x64, got = oracle.widen(host(xp)), oracle.widen(host(y))
    want = np.full((T * k, d), 7.0)
    for e in range(E):
        lo, hi = int(off[e]), int(off[e + 1])
        if hi > lo:
            want[lo:hi] = oracle.ffn_rows(x64[lo:hi], *(oracle.widen(host(w[e])) for w in (wg, wu, wd)), threads=8)
    return got, want, off


def check_segments(got, want, off, tol):
    for lo, hi in zip(off[:-1], off[1:]):
        if hi > lo:
            assert rel_err(got[lo:hi], want[lo:hi]) <= tol, (lo, hi)
    np.testing.assert_array_equal(got[off[-1]:], want[off[-1]:])   # rows of no segment keep what they held


@pytest.mark.parametrize("seg_rows,T,k,d,f", [
    ([1], 1, 1, 2048, 1024),                        # one row: 16 wavefronts share K
    ([0, 1, 0, 3], 4, 1, 136, 200),                 # K of 4 whole steps and 8 left over; strips past N in both projections
    ([16, 15, 0, 1], 16, 4, 256, 96),               # full and nearly full fragment of 16 rows; fewer K steps than the ring is deep
    ([17, 31, 32], 32, 3, 512, 352),                # two fragments
    ([33, 48, 49, 64], 64, 4, 1024, 768),           # three and four fragments
    ([64, 130, 5], 64, 4, 192, 72),                 # more rows in a segment than tokens: walked in pieces
    ([40, 30], 64, 2, 2048, 352),                   # few strips and long K: as many wavefronts as 64 KB of LDS allow
    ([20, 40], 20, 3, 4096, 40),                    # the same with two fragments; long K up, K of one step and a rest down
])
def test_few_rows_per_segment(seg_rows, T, k, d, f):
    """The weight-streaming kernel of decode batches (at most 64 tokens)."""
    assert kernels_of(T, k, d, f, len(seg_rows), len(seg_rows)) == ("stream", "stream")
    got, want, off = ffn_of_segments(seg_rows, T, k, d, f)
    check_segments(got, want, off, TOL["bf16"])


@pytest.mark.parametrize("seg_rows,T,k,d,f", [
    ([1], 70, 1, 2048, 1024),                       # one row, long K
    ([0, 1, 0, 3, 16, 17, 33], 70, 2, 136, 200),    # K of whole steps and 8 left over; strips past N
    ([32, 33, 64, 65, 96, 97], 97, 4, 192, 72),     # edges of the pieces of two, four and six fragments
    ([0, 200, 300], 300, 2, 448, 352),              # several pieces; K of half a step, fewer steps than are loaded ahead
    ([100, 40], 100, 2, 64, 8),                     # K of one step up, of 8 down
    ([130, 7], 130, 2, 8, 64),
    ([2] * 70 + [150, 1], 150, 4, 64, 40),          # more segments than lanes
])
def test_ordinary_batches(seg_rows, T, k, d, f):
    """The kernel between decode batches and large tiles."""
    assert kernels_of(T, k, d, f, len(seg_rows), len(seg_rows)) == ("mid", "mid")
    got, want, off = ffn_of_segments(seg_rows, T, k, d, f)
    check_segments(got, want, off, TOL["bf16"])


@pytest.mark.parametrize("seg_rows,T,k,d,f", [
    ([96 * 256], 24576, 1, 72, 64),                 # a tile per compute unit: none is cut
    ([96 * 256 + 1], 24577, 1, 72, 64),             # one tile of one row in halves; the down projection's second half past N
    ([96 * 384 - 40], 36824, 1, 72, 40),            # the second ones of half the units; gate+up halves of 32 and 8 columns
    ([96 * 384 + 1], 36865, 1, 72, 64),             # one more: none is cut
    ([96 * 511 - 40], 49016, 1, 72, 40),            # nor with all but one of the second ones
    ([96 * 512], 49152, 1, 72, 64),                 # two tiles each: none is cut
    ([1, 96, 97, 0, 50, 33, 32, 16] * 2 + [70, 64, 17, 200], 200, 20, 2056, 968),   # ragged last strips, 340 and 357 tiles
    ([3, 0, 40, 90, 17] * 26, 90, 44, 264, 136),    # more segments than lanes
    ([96 * 128], 12288, 1, 72, 64),                 # a half per compute unit, pieces of 96 rows
    ([48 * 128, 0], 6144, 1, 72, 64),               # of 48
    ([48 * 128 - 31, 1], 6144, 1, 72, 40),          # one too many for that in both projections: of 96; ragged halves
    ([32 * 128], 4096, 1, 72, 64),                  # of 32
    ([33, 0, 31, 65, 1], 66, 2, 1032, 328),         # of 32; half strips past N in both projections
])
def test_tiles_in_halves(seg_rows, T, k, d, f):
    """Between one tile and one and a half per compute unit of a 256-unit GPU: those past the first per unit are halved.  Few
    tiles: all are, in pieces of 32, 48 or 96 rows."""
    assert kernels_of(T, k, d, f, len(seg_rows), len(seg_rows)) == ("mid", "mid")
    got, want, off = ffn_of_segments(seg_rows, T, k, d, f)
    check_segments(got, want, off, TOL["bf16"])


@pytest.mark.parametrize("T,k,d,f,dtype,down", [
    (3, 2, 64, 32, "bf16", "stream"), (40, 4, 256, 128, "f32", "stream"), (130, 4, 200, 72, "bf16", "mid"), (90, 4, 40, 24, "f32", "stream"),
    (90, 4, 100, 50, "f32", "vector_f32"), (3000, 8, 256, 512, "bf16", "mid"), (25000, 2, 256, 128, "bf16", "persist"),
    (6000, 8, 1280, 640, "f32", "mid"), (3, 2, 8, 8388616, "bf16", "generic")])
def test_fresh_output_is_zero_outside_the_rank(T, k, d, f, dtype, down):
    """Every kernel's down projection zeroes what it does not compute of a y that holds NaN: rows before and behind the rank's, for
    a rank without rows all; the rank's rows are those of the call on zeros."""
    assert kernels_of(T, k, d, f, 2, 8, dtype=dtype)[1] == down
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(T)
    table = grace.GraceTable(8, 4, 1, [0] * 4, [1] * 4, list(range(9)), [e // 2 for e in range(8)])
    w = [(torch.randn(s, generator=gen, device="cuda") * 0.1).to(tdt) for s in ((2, f, d), (2, f, d), (2, d, f))]
    x = torch.randn((T * k, d), generator=gen, device="cuda").to(tdt)
    cuts = [0, 0, T * k // 5, T * k // 3, T * k // 2, T * k // 2, T * k // 2, T * k - 1, T * k]
    off = torch.tensor(cuts, dtype=torch.int32, device="cuda")
    ws = torch.empty(grace.grace_workspace_bytes(T, 8, k, 8, d, f, 0, int(dtype == "bf16")), dtype=torch.uint8, device="cuda")
    for rank in range(4):
        want = torch.zeros_like(x)
        grace.grace_expert_ffn(table, rank, x, off, T, k, *w, y=want)
        y = torch.full_like(x, float("nan"))
        grace.grace_expert_ffn_up(table, rank, x, off, T, k, w[0], w[1], ws)
        grace.grace_expert_ffn_down_fresh(table, rank, off, T, k, w[2], y, ws)
        assert torch.equal(y, want) and torch.equal(grace.grace_expert_ffn(table, rank, x, off, T, k, *w), want)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T,k,d,f", [(1, 1, 8, 8), (37, 3, 136, 64), (3000, 8, 2048, 64)])
def test_rank_without_instances_gives_zeros(T, k, d, f, dtype):
    """A table may leave a rank without instances; its call then has nothing to read of the weights, which need not be empty, and
    all rows are other ranks'.  The buffer that torch hands out here held NaN."""
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    table = grace.GraceTable(2, 3, 1, [0] * 3, [1] * 3, [0, 1, 2], [0, 2])
    assert len(table.local_experts(1)) == 0
    off = torch.tensor([0, T * k // 2, T * k], dtype=torch.int32, device="cuda")
    x = torch.ones((T * k, d), dtype=tdt, device="cuda")
    w = [torch.ones(s, dtype=tdt, device="cuda") for s in ((1, f, d), (1, f, d), (1, d, f))]
    ws = torch.empty(grace.grace_workspace_bytes(T, 2, k, 2, d, f, 0, int(dtype == "bf16")), dtype=torch.uint8, device="cuda")
    y = torch.full_like(x, float("nan"))
    grace.grace_expert_ffn_down_fresh(table, 1, off, T, k, w[2], y, ws)
    assert torch.equal(y, torch.zeros_like(y))
    torch.cuda.empty_cache()
    held = torch.full_like(x, float("nan"))
    del held
    assert torch.equal(grace.grace_expert_ffn(table, 1, x, off, T, k, *w, ws=ws), torch.zeros_like(x))


@pytest.mark.parametrize("T,k,d,f,S,I,dtype,up,threads", [
    (3000, 8, 200, 1032, 1, 64, "bf16", True, 256),
    (3000, 8, 200, 1032, 1, 64, "bf16", False, 256),
    (200, 8, 1024, 2048, 8, 64, "f32", True, 256),
    (1000, 8, 8192, 640, 8, 64, "f32", False, 256),
    (400, 8, 1024, 1024, 8, 128, "f32", False, 512),    # two groups of wavefronts share K
])
def test_more_rows_than_a_rank_is_expected_to_hold(T, k, d, f, S, I, dtype, up, threads):
    """The 96-row and the split kernels' grids cover five times a rank's even share; here one rank of many holds every row, so that
    workgroups take several tiles."""
    dt, tile_rows = (grace.GRACE_F32, 80) if dtype == "f32" else (grace.GRACE_BF16, 96)
    seg_rows = [T * k // S] * S
    kernel, items = grace.grace_ffn_kernel(up, T, d, f, dt, k=k, S=S, I=I)
    strips = -(-f // 64) if up else -(-d // 128)
    assert kernel == "mid" and items < S * -(-seg_rows[0] // tile_rows) * strips * threads     # fewer workgroups than whole tiles
    ffn_rows_of_segments(seg_rows, T, k, d, f, dtype, first=8, I=I, S=S)


def test_up_projection_of_decode_batches():
    """More than 16 tokens whose gate+up strips fill the chip: streaming kernel for the down projection only."""
    assert kernels_of(40, 2, 256, 16 * 1024 + 24, 4, 4) == ("mid", "stream")
    got, want, off = ffn_of_segments([17, 0, 40, 9], 40, 2, 256, 16 * 1024 + 24)
    check_segments(got, want, off, TOL["bf16"])


def test_large_tiles():
    """Large batches keep the 256 x 256 tiles (the gate+up projection here)."""
    assert kernels_of(5000, 1, 128, 2048, 4, 4) == ("persist", "mid")
    got, want, off = ffn_of_segments([4700, 0, 257, 43], 5000, 1, 128, 2048)
    check_segments(got, want, off, TOL["bf16"])


@pytest.mark.parametrize("seg_rows,T,k,d,f,want", [
    ([1, 0, 2], 3, 1, 1024, 256, ("stream", "stream")),          # few rows: one workgroup per strip and segment
    ([40, 0, 25], 64, 2, 100, 76, ("stream", "stream")),         # K of 6 whole steps and 4 left over; strips past N
    ([65, 64, 0, 1], 65, 2, 128, 256, ("stream", "stream")),     # pieces: 65 rows in two, one full, one row
    ([0, 130, 17, 300], 300, 2, 180, 260, ("stream", "stream")),    # pieces of one, two and three fragments with ragged ends
    ([33, 97], 100, 2, 36, 77, ("stream", "vector_f32")),        # odd N up; the down projection's K takes the vector kernel
    ([33, 97], 100, 2, 34, 64, ("vector_f32", "stream")),        # odd N down
    ([1] * 70 + [80] * 3, 160, 2, 64, 32, ("stream", "stream")),    # more segments than lanes
    ([1] * 70 + [80] * 3, 160, 2, 36, 77, ("stream", "vector_f32")),
    ([1, 0] * 40, 40, 1, 64, 48, ("stream", "stream")),          # the same with one workgroup per strip and segment
])
def test_f32_segments(seg_rows, T, k, d, f, want):
    """fp32 streaming kernel: one workgroup per strip (at most 64 tokens) or per strip and piece of a segment."""
    assert kernels_of(T, k, d, f, len(seg_rows), len(seg_rows), dtype="f32") == want
    got, ref, off = ffn_of_segments(seg_rows, T, k, d, f, torch.float32)
    check_segments(got, ref, off, TOL["f32"])


def ffn_rows_of_segments(seg_rows, T, k, d, f, dt, first=0, I=None, S=None):
    """Expert FFN of the rank that hosts instances `first` .. `first + S - 1` of I, all segments of that rank, and the oracle's
    result for some rows of each segment: both ends, the first pieces' edges and a few more."""
    S, I = S or len(seg_rows), I or len(seg_rows)
    tdt = torch.bfloat16 if dt == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(sum(seg_rows))
    rng = np.random.default_rng(sum(seg_rows))

    def normal(scale, *shape):
        return (scale * torch.randn(shape, generator=gen, device="cuda")).to(tdt)

    R = I // S
    table = grace.GraceTable(I, R, 1, [0] * R, [1] * R, list(range(I + 1)), [e // S for e in range(I)])
    w = normal(0.05, S, f, d), normal(0.05, S, f, d), normal(0.05, S, d, f)
    x = normal(1.0, T * k, d)
    off = np.zeros(I + 1, dtype=np.int32)
    off[first + 1:first + S + 1] = np.cumsum(seg_rows)
    off[first + S + 1:] = off[first + S]
    y = grace.grace_expert_ffn(table, first // S, x, torch.from_numpy(off).cuda(), T, k, *w)
    assert not y[int(off[first + S]):].any()
    for s in range(S):
        lo, hi = int(off[first + s]), int(off[first + s + 1])
        if hi == lo:
            continue
        rows = np.unique(np.clip([lo, hi - 1, lo + 15, lo + 16, lo + 95, lo + 96, *(lo + rng.integers(0, hi - lo, 10))], lo, hi - 1))
        ref = oracle.ffn_rows(oracle.widen(host(x[rows])), *(oracle.widen(host(m[s])) for m in w), threads=8)
        assert rel_err(oracle.widen(host(y[rows])), ref) <= TOL[dt], (s, lo, hi)


@pytest.mark.parametrize("seg_rows,T,k,d,f,want", [
    ([1, 0, 17, 33, 49, 65, 81, 96], 96, 8, 1024, 2048, ("mid", "mid")),       # pieces of one to five fragments
    ([1, 0, 0, 0, 0, 0, 0, 2], 65, 2, 1028, 2052, ("mid", "mid")),             # few tiles, of 16 rows; K and N off the steps
    ([40, 0, 0, 0, 0, 0, 0, 24], 65, 2, 1024, 2048, ("mid", "stream")),        # of 32
    ([130, 0, 0, 0, 0, 0, 0, 0], 130, 2, 1024, 2048, ("mid", "mid")),          # of 32 and 48, half the weight rows
    ([300, 0, 0, 0, 0, 0, 50, 0], 300, 2, 1024, 2048, ("mid", "mid")),         # of 80
    ([0, 3000, 1, 97, 1500, 95, 700, 807], 3100, 2, 1284, 644, ("mid", "mid")),    # long launches; K and N off the steps and strips
    ([0, 1, 95, 96, 97] * 14 + [2154], 6200, 1, 1280, 640, ("mid", "mid")),    # more segments than lanes
])
def test_f32_long_launches(seg_rows, T, k, d, f, want):
    """fp32 in tiles of up to 80 rows and 128 weight rows."""
    assert kernels_of(T, k, d, f, len(seg_rows), len(seg_rows), dtype="f32") == want
    ffn_rows_of_segments(seg_rows, T, k, d, f, "f32")


@pytest.mark.parametrize("seg_rows,N", [([193, 1], 32 * 12), ([65, 33], 32 * 21), ([65, 33], 32 * 22), ([65, 33], 32 * 42), ([65, 33], 32 * 43)])
def test_f32_pieces_of_16_and_32_rows(seg_rows, N):
    """Tiles of 64 rows on a quarter and half of the compute units (256), and one strip more: pieces of 16, 32 and 64 rows."""
    T, f = max(seg_rows), 68
    assert kernels_of(T, 2, N, f, 2, 2, dtype="f32")[1] == "stream"
    ffn_rows_of_segments(seg_rows, T, 2, N, f, "f32")


@pytest.mark.parametrize("seg_rows,T,k,d,f,want", [
    ([16, 17, 33, 49, 65, 80, 81, 161], 260, 2, 516, 515, ("mid", "vector_f32")),     # pieces of one to five fragments; N no multiple of 4; K of 16 steps and 4
    ([120, 0, 1, 70, 3, 9, 200, 64], 250, 2, 1024, 1100, ("mid", "mid")),      # down: few tiles, the groups share a K of 34 steps and 12
    ([90, 300, 10, 0, 0, 0, 0, 0], 210, 2, 2052, 2820, ("mid", "mid")),        # an odd number of steps
    ([70] * 70, 2500, 2, 512, 1024, ("mid", "mid")),                           # more segments than lanes
])
@pytest.mark.parametrize("scale", [1.0, 1e-15, 1e20])          # inside the split's range and on either side of it
def test_f32_split_kernel(seg_rows, T, k, d, f, want, scale):
    assert kernels_of(T, k, d, f, len(seg_rows), len(seg_rows), dtype="f32") == want
    if scale != 1.0 and len(seg_rows) > 8:
        pytest.skip("the range does not depend on the number of segments")
    S = len(seg_rows)
    gen = torch.Generator(device="cuda").manual_seed(T)
    table = grace.GraceTable(S, 1, 1, [0], [1], list(range(S + 1)), [0] * S)
    x = scale * torch.randn((T * k, d), generator=gen, device="cuda")
    wg, wu, wd = (0.05 * torch.randn(n, generator=gen, device="cuda") for n in ((S, f, d), (S, f, d), (S, d, f)))
    if scale > 1.0:
        wu /= scale   # (the hidden activation stays finite)
    off = np.concatenate([[0], np.cumsum(seg_rows)]).astype(np.int32)
    y = grace.grace_expert_ffn(table, 0, x, torch.from_numpy(off).cuda(), T, k, wg, wu, wd)
    for s in range(S):
        if off[s] == off[s + 1]:
            continue
        xs = x[off[s]:off[s + 1]].double()
        h = torch.nn.functional.silu(xs @ wg[s].double().T) * (xs @ wu[s].double().T)
        ref = h @ wd[s].double().T
        assert rel_err(y[off[s]:off[s + 1]].cpu().numpy().astype(np.float64), ref.cpu().numpy()) <= TOL["f32"], s


def test_f32_split_kernel_infinities_and_nans():
    """An infinity or a NaN in one row: that row is what fp32 arithmetic gives, the others are as without it."""
    T, d, f = 900, 1024, 2816
    gen = torch.Generator(device="cuda").manual_seed(3)
    table = grace.GraceTable(1, 1, 1, [0], [1], [0, 1], [0])
    x = torch.randn((T, d), generator=gen, device="cuda")
    wg, wu, wd = (0.05 * torch.rand(n, generator=gen, device="cuda") for n in ((1, f, d), (1, f, d), (1, d, f)))
    off = torch.tensor([0, T], dtype=torch.int32, device="cuda")
    plain = grace.grace_expert_ffn(table, 0, x, off, T, 1, wg, wu, wd)
    x[7, 100] = float("inf")
    x[90, 3] = float("nan")
    x[150] = 0.0
    y = grace.grace_expert_ffn(table, 0, x, off, T, 1, wg, wu, wd)
    assert kernels_of(T, 1, d, f, 1, 1, dtype="f32") == ("mid", "mid")
    assert torch.isposinf(y[7]).all() and torch.isnan(y[90]).all() and not y[150].any()
    rest = [i for i in range(T) if i not in (7, 90, 150)]
    assert rel_err(y[rest].cpu().numpy().astype(np.float64), plain[rest].cpu().numpy().astype(np.float64)) <= TOL["f32"]


def test_f32_split_rows_do_not_depend_on_their_neighbours():
    """Bit for bit the same row whatever else is in the batch: few rows (half tiles, low pieces) or many (whole tiles), ordinary ones or such
    as are computed without the split."""
    T, k, d, f = 1000, 2, 1024, 2816
    few, many = [40, 3, 1, 0], [700, 600, 300, 400]
    assert kernels_of(T, k, d, f, 4, 4, dtype="f32") == ("mid", "mid")
    gen = torch.Generator(device="cuda").manual_seed(11)
    table = grace.GraceTable(4, 1, 1, [0], [1], list(range(5)), [0] * 4)
    w = [0.05 * torch.randn(s, generator=gen, device="cuda") for s in ((4, f, d), (4, f, d), (4, d, f))]
    w[0][1, 7, 5] = 1e-36      # (one of a column's values: that column alone is affected, if any)
    x = torch.randn((T * k, d), generator=gen, device="cuda")
    first = np.concatenate([[0], np.cumsum(many)])
    y = []
    for segs, odd in ((few, False), (many, False), (many, True)):
        off = np.concatenate([[0], np.cumsum(segs)]).astype(np.int32)
        xs = x.clone()
        for s in range(4):
            xs[off[s]:off[s] + few[s]] = x[first[s]:first[s] + few[s]]
            if odd:
                xs[off[s] + few[s]:off[s + 1]:3] = torch.tensor([1e-30, 1e25, float("inf"), float("nan")][s], device="cuda")
        out = grace.grace_expert_ffn(table, 0, xs, torch.from_numpy(off).cuda(), T, k, *w)
        y.append(torch.cat([out[off[s]:off[s] + few[s]] for s in range(4)]))
    assert torch.equal(y[0], y[1]) and torch.equal(y[0], y[2])


def test_f32_split_keeps_small_values_of_a_row_with_large_ones():
    """An element of 2^-120 next to 1: its lowest parts lie below the range of bf16, and it is all that its column sees."""
    T, d, f = 1000, 1024, 1024
    assert kernels_of(T, 1, d, f, 1, 1, dtype="f32")[0] == "mid"
    gen = torch.Generator(device="cuda").manual_seed(5)
    table = grace.GraceTable(1, 1, 1, [0], [1], [0, 1], [0])
    x = torch.zeros((T, d), device="cuda")
    x[:, 0] = 1.0
    x[:, 1] = 2.0 ** -120 * (1.0 + torch.rand(T, generator=gen, device="cuda"))
    wg, wu, wd = (torch.randn(s, generator=gen, device="cuda") for s in ((1, f, d), (1, f, d), (1, d, f)))
    wg[0, :, 0] = 0.0
    wg[0, :, 1] = 2.0 ** 30 * (1.0 + torch.rand(f, generator=gen, device="cuda"))
    wu[0, :, 0] *= 2.0 ** 50
    y = grace.grace_expert_ffn(table, 0, x, torch.tensor([0, T], dtype=torch.int32, device="cuda"), T, 1, wg, wu, wd)
    h = torch.nn.functional.silu(x.double() @ wg[0].double().T) * (x.double() @ wu[0].double().T)
    assert rel_err(y.cpu().numpy().astype(np.float64), (h @ wd[0].double().T).cpu().numpy()) <= TOL["f32"]   # (1.3e-6; 5.9e-5 without)


@pytest.mark.parametrize("T,d", [(97, 520), (7000, 520), (90, 515)])     # both numbers of groups that share K; rows of no whole vectors
@pytest.mark.parametrize("odd", ["small", "infinite"])
def test_f32_split_of_segmented_k_out_of_range(T, d, odd):
    """Shared experts' down projection, K segments off the step: sums too small for the split, and infinities among the weights."""
    f, n_shared = 200, 3
    assert kernels_of(T, 1, d, f, 1, 1, n_shared=n_shared, dtype="f32")[1] == "mid"
    gen = torch.Generator(device="cuda").manual_seed(T)
    x = torch.randn((T, d), generator=gen, device="cuda") * (1e-14 if odd == "small" else 1.0)
    wg, wu, wd = (0.05 * torch.randn(s, generator=gen, device="cuda") for s in ((n_shared, f, d), (n_shared, f, d), (n_shared, d, f)))
    if odd == "infinite":
        wd[1, 17, 150] = float("inf")
    y = grace.grace_shared_ffn(x, wg, wu, wd).cpu().numpy().astype(np.float64)
    want = 0.0
    for s in range(n_shared):
        h = torch.nn.functional.silu(x.double() @ wg[s].double().T) * (x.double() @ wu[s].double().T)
        want = want + h @ wd[s].double().T
    want = want.cpu().numpy()
    if odd == "infinite":
        assert (y[:, 17] == want[:, 17]).all() and np.isinf(y[:, 17]).all()
        y, want = np.delete(y, 17, axis=1), np.delete(want, 17, axis=1)
    assert rel_err(y, want) <= TOL["f32"]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T,d,f,n_shared", [(1, 2048, 1408, 2), (64, 512, 96, 3), (33, 136, 200, 2), (97, 520, 40, 3),
                                            (1100, 1024, 200, 3),    # 12 pieces x 8 strips: more than one tile per run of an XCD
                                            (1900, 2056, 104, 2)])   # 20 x 17 tiles: the second ones in halves
def test_shared_experts_small_batches(T, d, f, n_shared, dtype):
    """Shared experts: the down projection's K runs through n_shared segments (lengths below, at and off the K step);
    the row scatter is a launch of its own here."""
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    rng = np.random.default_rng(T)

    def normal(scale, *shape):
        return torch.from_numpy((scale * rng.standard_normal(shape)).astype(np.float32)).cuda().to(tdt)

    x, wg, wu, wd = normal(1.0, T, d), normal(0.05, n_shared, f, d), normal(0.05, n_shared, f, d), normal(0.05, n_shared, d, f)
    got = grace.grace_shared_ffn(x, wg, wu, wd)
    pos = torch.from_numpy(rng.permutation(T * 2).astype(np.int32)).cuda()
    ws = torch.zeros(grace.grace_workspace_bytes(T, 1, 1, 1, d, f, n_shared, grace.GRACE_F32 if dtype == "f32" else grace.GRACE_BF16),
                     dtype=torch.uint8, device="cuda")
    xp = torch.zeros((T * 2, d), dtype=tdt, device="cuda")
    grace.grace_shared_ffn_up_scatter(x, wg, wu, ws, pos, 2, xp)
    two = grace.grace_shared_ffn_down(wd, ws, T)
    torch.cuda.synchronize()
    want = oracle.shared_ffn(oracle.widen(host(x)), tuple(oracle.widen(host(w)) for w in (wg, wu, wd)), threads=8)
    assert rel_err(oracle.widen(host(got)), want) <= TOL[dtype]
    assert torch.equal(got, two)
    np.testing.assert_array_equal(host(xp)[pos.cpu().numpy()], np.repeat(host(x), 2, axis=0))


@pytest.mark.parametrize("T,k,dtype", [(1, 1, "bf16"), (7, 2, "f32"), (33, 3, "bf16"), (5, 5, "bf16"), (1024, 6, "f32"), (1025, 9, "bf16")])
def test_combine_with_absent_rows(T, k, dtype):
    """Choices loaded ahead, with positions outside the buffer (no row) among them and NaN in a row nobody names."""
    rng = np.random.default_rng(T * k)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    y = torch.from_numpy(rng.standard_normal((T * k, 24)).astype(np.float32)).to(tdt)
    pos = rng.permutation(T * k).astype(np.int32)
    pos[rng.random(T * k) < 0.3] = -1
    pos[pos == 0] = T * k
    y[0] = float("nan")
    w = rng.random((T, k)).astype(np.float32)
    out = grace.grace_combine(y.cuda(), torch.from_numpy(pos).cuda(), torch.from_numpy(w).cuda())
    got, rows = oracle.widen(host(out)), oracle.widen(host(y))
    want = np.zeros((T, 24))
    for a, p in enumerate(pos):
        if 0 <= p < T * k:
            want[a // k] += np.float64(w.reshape(-1)[a]) * rows[p]
    assert rel_err(got, want) <= (1e-6 if dtype == "f32" else 2.0 ** -8)   # one rounding of an fp32 sum


@pytest.mark.parametrize("T,k,d,dtype,lo,hi,shared", [
    (1, 1, 24, "bf16", 0, 1, False), (1, 8, 2056, "bf16", 2, 3, True), (5, 70, 24, "f32", 60, 300, False), (300, 70, 24, "f32", 6000, 15000, False),
    (33, 64, 24, "bf16", 3, 700, True), (1024, 6, 24, "f32", 0, 0, True), (1025, 9, 24, "bf16", 1000, 4000, True), (1027, 16, 2056, "bf16", 0, 16432, False),
    (1025, 17, 24, "f32", 9000, 17425, False), (2051, 2, 1028, "f32", 4101, 4102, True),
    (3, 2, 2048, "bf16", 1, 4, True), (40, 3, 4096, "bf16", 30, 90, False), (40, 2, 4104, "bf16", 0, 60, True), (5, 70, 2052, "f32", 60, 300, True), (2049, 3, 2056, "bf16", 900, 2100, True)])   # one or more passes of a workgroup over a row
def test_combine_share_is_combine_of_zero_rows(T, k, d, dtype, lo, hi, shared):
    """Rows outside the share are zero and not read: the same bits as grace_combine, which reads them, with positions
    outside the buffer and gate weights that are not finite (0 * inf) among the absent rows."""
    rng = np.random.default_rng(T + k)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    y = torch.zeros((T * k, d), dtype=tdt, device="cuda")
    y[lo:hi] = torch.from_numpy(rng.standard_normal((hi - lo, d)).astype(np.float32)).cuda().to(tdt)
    pos = rng.permutation(T * k).astype(np.int32)
    pos[rng.random(T * k) < 0.1] = -1
    pos[rng.random(T * k) < 0.1] = T * k
    w = rng.random((T, k)).astype(np.float32)
    w[rng.random((T, k)) < 0.02] = np.inf
    ys = torch.from_numpy(rng.standard_normal((T, d)).astype(np.float32)).cuda().to(tdt) if shared else None
    state = torch.tensor([5, 9, 0, 0, lo, hi, 0, 0], dtype=torch.int32, device="cuda")
    pos, w = torch.from_numpy(pos).cuda(), torch.from_numpy(w).cuda()
    want = grace.grace_combine(y, pos, w, ys)
    y[:lo] = 3.0   # not read
    y[hi:] = 3.0
    got = grace.grace_combine_share(y, pos, w, state, ys)
    torch.testing.assert_close(got, want, rtol=0, atol=0, equal_nan=True)


@pytest.mark.parametrize("R", [1, 2])
def test_combine_of_a_layer_that_hosts_every_instance(R):
    """Nothing to leave out: grace_combine, with the bits of grace_combine_share."""
    T, E, k, d, f = 33, 8, 2, 72, 40
    gen = torch.Generator(device="cuda").manual_seed(R)
    table = grace.GraceTable(E, R, 1, [0] * R, [1] * R, list(range(E + 1)), [e * R // E for e in range(E)])
    S = E // R
    w = [(torch.randn(s, generator=gen, device="cuda") * 0.1).bfloat16() for s in ((S, f, d), (S, f, d), (S, d, f))]
    layer = grace.GraceMoELayer(table, 0, T, k, d, f, torch.bfloat16, *w)
    out = layer.forward(torch.randn((T, E), generator=gen, device="cuda"), torch.randn((T, d), generator=gen, device="cuda").bfloat16())
    lib = grace.load_library()
    assert layer._calls[-1][1] is (lib.grace_combine if R == 1 else lib.grace_combine_share)
    assert torch.equal(out, grace.grace_combine_share(layer.y, layer.perm_out[0], layer.route_out[1], layer.y_state))


@pytest.mark.parametrize("T,E,k,d,dtype,rows,policy", [
    (1, 1, 1, 8, "bf16", True, 0), (1, 256, 64, 2048, "f32", True, 1), (2, 64, 8, 2048, "bf16", True, 0),
    (4, 65, 3, 4, "f32", True, 0), (5, 128, 8, 24, "bf16", True, 1), (16, 129, 8, 4096, "bf16", True, 0),
    (17, 200, 60, 8, "bf16", False, 0), (33, 60, 4, 2056, "bf16", False, 1), (63, 193, 16, 40, "f32", True, 0),
    (64, 64, 16, 9000, "bf16", True, 0),    # rows of more vectors than a workgroup has threads
    (65, 64, 8, 8, "bf16", True, 0), (32, 128, 8, 2048, "bf16", True, 0), (31, 256, 8, 40, "f32", True, 1), (96, 8, 4, 128, "f32", True, 1), (256, 8, 2, 128, "f32", True, 0),
    (64, 64, 17, 8, "bf16", True, 0), (97, 64, 3, 8, "bf16", True, 0), (257, 64, 2, 8, "bf16", True, 0), (33, 65, 3, 8, "bf16", True, 0)])   # past it, in assignments and in tokens
def test_one_launch_dispatch_of_few_tokens(T, E, k, d, dtype, rows, policy):
    """Routing, index work and rows of up to 96 (k = 2: 256) tokens in one launch against the oracle and, bit for bit, the separate
    calls: ties, masked experts, counters near 2^32, experts with several candidates."""
    rng = np.random.default_rng(T * E + k)
    R = 4
    hosts = [sorted(rng.choice(R, size=1 if E > 200 else rng.integers(1, 4 if E < 80 else 2), replace=False).tolist()) for _ in range(E)]
    ptr = np.concatenate([[0], np.cumsum([len(h) for h in hosts])])
    assert ptr[-1] <= 256
    pl = SimpleNamespace(E=E, R=R, N=2, rank_node=np.array([0, 0, 1, 1], np.int32), poll_weight=rng.integers(1, 9, size=R).astype(np.uint32),
                         inst_ptr=ptr.astype(np.int32), inst_rank=np.concatenate(hosts).astype(np.int32))
    table = grace.GraceTable.from_placement(pl)
    logits = np.round(rng.standard_normal((T, E)) * 2).astype(np.float32) / 2
    logits[0, ::2] = -0.0
    logits[T // 2, 1:] = -np.inf
    logits_host = logits
    logits = torch.from_numpy(logits).cuda()
    x = torch.from_numpy(rng.standard_normal((T, d)).astype(np.float32)).cuda().to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    rr = torch.from_numpy(rng.integers(2 ** 32 - 9, 2 ** 32, size=E, dtype=np.uint64).astype(np.uint32).view(np.int32)).cuda()
    out_a, out_b = torch.zeros_like(rr), torch.zeros_like(rr)
    route = grace.grace_route(table, 2, logits, k, 0, rr, out_a, policy=policy)
    perm = grace.grace_permute(table, route[2], x if rows else None)
    one = grace.grace_route_permute(table, 2, logits, k, x if rows else None, 0, rr, out_b, policy=policy)
    for a, b in zip((*route, *perm, out_a), (*one[0], *one[1], out_b)):
        assert (a is None and b is None) or torch.equal(a, b)
    ref = oracle.route_permute(logits_host, pl, k, 2, renorm=0, rr_in=rr.cpu().numpy().view(np.uint32), policy=policy)
    (te, tw, ti, cnt), (pos, src, ioff, roff, noff, xp) = one
    parity.check_route_permute(SimpleNamespace(te=te, tw=tw, ti=ti, cnt=cnt, rout=out_b, pos=pos, src=src, ioff=ioff, roff=roff, noff=noff, xp=xp),
                               ref, SimpleNamespace(x=host(x)), k)


@pytest.mark.parametrize("nodes,gpus,T,k", [(2, 2, 1, 2), (3, 2, 255, 4), (1, 4, 1025, 3), (4, 2, 513, 2)])
def test_send_list_block_edges(nodes, gpus, T, k):
    """Send lists whose assignments end just below, at and past a block of the counting and the expansion kernels."""
    E, R = 16, nodes * gpus
    rng = np.random.default_rng(T)
    ranks = [e % R for e in range(E)]
    table = grace.GraceTable(E, R, nodes, [r // gpus for r in range(R)], [1] * R, list(range(E + 1)), ranks)
    experts = np.stack([rng.permutation(E)[:k] for _ in range(T)])
    order = sorted(range(E), key=lambda e: (ranks[e], e))
    inst = np.empty(E, np.int32)
    inst[order] = np.arange(E, dtype=np.int32)
    topk_inst = torch.from_numpy(inst[experts].astype(np.int32)).cuda()
    rp, rt, np_, nt, ex, tr = (t.cpu().numpy() for t in grace.grace_send_lists(table, R - 1, topk_inst))
    dest = np.array(ranks)[experts]
    for r in range(R):
        np.testing.assert_array_equal(rt[rp[r]:rp[r + 1]], np.flatnonzero((dest == r).any(axis=1)))
    for n in range(nodes):
        np.testing.assert_array_equal(nt[np_[n]:np_[n + 1]], np.flatnonzero((dest // gpus == n).any(axis=1)))
    for a, d in enumerate(dest.reshape(-1)):
        assert rt[rp[d] + ex[a]] == a // k
    other = (R - 1) // gpus
    assert tr[1] == int((dest // gpus != other).sum())
    assert tr[3] == int(((dest // gpus == other) & (dest != R - 1)).sum())


@pytest.mark.parametrize("R,T,k", [(1, 1, 1), (8, 1, 64), (5, 8, 64), (64, 170, 3), (512, 256, 2), (513, 256, 2), (6, 57, 9)])
def test_send_lists_in_one_workgroup(R, T, k):
    """At most 512 assignments and ranks in one launch: bit for bit the general kernels (separate scans), with several experts
    of a token on one rank, ids outside the table, and list entries past the ends."""
    nodes = max(1, R // 4)
    E = min(256, 2 * R)
    rng = np.random.default_rng(R + T)
    ptr, ranks = [0], []
    for e in range(E):
        ranks += sorted(rng.choice(R, size=min(R, int(rng.integers(1, 4))), replace=False).tolist())
        ptr.append(len(ranks))
    table = grace.GraceTable(E, R, nodes, [r * nodes // R for r in range(R)], [1] * R, ptr, ranks)
    ti = rng.integers(-2, table.I + 2, size=(T, k)).astype(np.int32)
    for local_rank in {0, R - 1}:
        got = [t.cpu().numpy() for t in grace.grace_send_lists(table, local_rank, torch.from_numpy(ti).cuda())]
        order = [t.cpu().numpy() for t in grace.grace_permute(table, torch.from_numpy(ti).cuda(), None)[:5]]
        table.set_fold_limits(0, 0)
        want = [t.cpu().numpy() for t in grace.grace_send_lists(table, local_rank, torch.from_numpy(ti).cuda())]
        order_want = [t.cpu().numpy() for t in grace.grace_permute(table, torch.from_numpy(ti).cuda(), None)[:5]]
        table.set_fold_limits()
        n_rows = int(order_want[2][-1])
        for g, w in zip(got, want):
            np.testing.assert_array_equal(g, w)
        assert (got[1][got[0][-1]:] == -1).all() and (got[3][got[2][-1]:] == -1).all()
        for i, (g, w) in enumerate(zip(order, order_want)):
            np.testing.assert_array_equal(g[:n_rows] if i == 1 else g, w[:n_rows] if i == 1 else w)


# ------------------------------------------- kernels that a test must reach, with the choice asserted --
def kernels_of(T, k, d, f, S, I, n_shared=0, dtype="bf16"):
    """Kernels of the gate+up and the down projection on the current device."""
    dt = grace.GRACE_F32 if dtype == "f32" else grace.GRACE_BF16
    return tuple(grace.grace_ffn_kernel(up, T, d, f, dt, k=k, S=S, I=I, n_shared=n_shared)[0] for up in (True, False))


@pytest.mark.parametrize("seg_rows,k,d,f,want", [
    ([300], 1, 128, 14336, ("persist", "mid")),       # 2 m-tiles x 112 n-tiles: pairs cut flat over the XCDs, the shortest K
    ([300], 1, 17408, 128, ("mid", "persist")),       # the same for the down projection, 2 x 68
    ([700], 1, 8704, 4096, ("persist", "persist")),   # fewer tiles than compute units, 136 and 64 K steps
    ([0, 1, 3] * 20 + [7] * 9 + [7857], 1, 512, 384, ("persist", "persist")),   # more segments than lanes, most of them a few rows
])
def test_large_tiles_of_few_and_of_many_segments(seg_rows, k, d, f, want):
    T, S = sum(seg_rows), len(seg_rows)
    assert kernels_of(T, k, d, f, S, S) == want
    got, ref, off = ffn_of_segments(seg_rows, T, k, d, f)
    check_segments(got, ref, off, TOL["bf16"])
    if S == 1:   # the shared experts' launches of the same shape
        rng = np.random.default_rng(T)
        x, wg, wu, wd = (torch.from_numpy((a * rng.standard_normal(n)).astype(np.float32)).cuda().to(torch.bfloat16)
                         for a, n in ((1.0, (T, d)), (0.05, (1, f, d)), (0.05, (1, f, d)), (0.05, (1, d, f))))
        assert kernels_of(T, 1, d, f, 1, 1, n_shared=1) == want
        y = grace.grace_shared_ffn(x, wg, wu, wd)
        ref = oracle.shared_ffn(oracle.widen(host(x)), tuple(oracle.widen(host(w)) for w in (wg, wu, wd)), threads=8)
        assert rel_err(oracle.widen(host(y)), ref) <= TOL["bf16"]


def test_operands_past_two_gigabytes():
    """K off 64 in rows so long that 128 of them pass 2 GB: no buffer loads, the 128 x 128 kernel."""
    T, d, f = 3, 8388616, 8
    assert kernels_of(T, 1, d, f, 1, 1)[0] == "generic"
    got, want, off = ffn_of_segments([T], T, 1, d, f)
    check_segments(got, want, off, TOL["bf16"])


@pytest.mark.parametrize("T,d,f,n_shared,k", [
    (3000, 512, 512, 2, 6),      # 1 KB rows, 12 row tiles x 8 column tiles of 8 K steps
    (1500, 512, 1024, 2, 64),    # the largest top-k: nearly all rows are moved after the tile loop
    (700, 2048, 1344, 3, 64),    # 4 KB rows, 3 x 32 tiles
    (1500, 4096, 2048, 1, 3),    # 8 KB rows, 6 x 16 tiles
    (1500, 512, 1024, 2, 65),    # more choices than a wavefront has lanes: the rows move in a launch of their own
])
def test_row_scatter_carried_by_the_large_tiles(T, d, f, n_shared, k):
    """grace_shared_ffn_up_scatter where the projection's launch moves the rows (k > 1, dropped positions)."""
    assert kernels_of(T, k, d, f, 1, 1, n_shared=n_shared)[0] == "persist"
    parity.test_shared_up_with_row_scatter_equals_the_two_calls(T, d, f, n_shared, k, "bf16")


@pytest.mark.parametrize("T,E,k,d,f,dtype,want", [
    (16, 8, 2, 256, 192, "bf16", ("stream", "stream")),
    (48, 32, 4, 256, 1024, "bf16", ("mid", "stream")),     # the record is written by one kernel, read by another
    (48, 80, 4, 1280, 320, "bf16", ("mid", "mid")),
    (200, 8, 2, 256, 192, "bf16", ("mid", "mid")),
    (20000, 8, 2, 128, 256, "bf16", ("persist", "mid")),
    (25000, 8, 2, 256, 128, "bf16", ("persist", "persist")),
    (40, 8, 2, 132, 100, "f32", ("stream", "stream")),     # fp32, one workgroup per strip
    (90, 8, 2, 100, 50, "f32", ("stream", "vector_f32")),
])
def test_rank_share_after_routing_changes_by_kernel(monkeypatch, T, E, k, d, f, dtype, want):
    """Rows of y that an earlier step wrote are zero after the rank's range has moved, whichever kernels run."""
    cfg = LayerConfig(f"{dtype}_share_{T}", T=T, E=E, k=k, d=d, f=f, dtype=dtype, zipf_s=0.5, nodes=1, gpus_per_node=2, n_hot=2,
                      replica_mode="all", seed=T)
    table = grace.GraceTable.from_placement(make_workload(cfg).placement)
    assert kernels_of(T, k, d, f, len(table.local_experts(1)), table.I, dtype=dtype) == want
    monkeypatch.setitem(parity.SMALL, cfg.name, cfg)
    parity.test_layer_rank_share_after_routing_changes(cfg.name)


@pytest.mark.parametrize("T,k,d,f,S,I,dtype,want", [
    (3000, 8, 2048, 1024, 18, 72, "bf16", "persist"),    # ragged tiles, some with an idle half; idle workgroups in the last round move the rows
    (12000, 2, 512, 1024, 4, 16, "bf16", "persist"),     # k = 2, a piece per row
    (9000, 8, 512, 256, 90, 90, "bf16", "persist"),      # more segments than lanes; every row is the rank's
    (6000, 8, 512, 384, 8, 16, "bf16", "persist"),
    (2100, 17, 1024, 512, 8, 8, "bf16", "persist"),
    (40, 4, 512, 256, 4, 8, "bf16", "stream"),           # other kernels: the rows move in a launch of their own
    (3000, 8, 544, 256, 8, 16, "bf16", None),            # rows that are no whole 1 KB pieces
    (90, 2, 512, 256, 4, 8, "f32", "stream"),
])
def test_gate_up_projection_that_moves_the_rows(T, k, d, f, S, I, dtype, want):
    """Bit for bit the row scatter and then the projection on the moved rows; ids outside the table leave no row."""
    kernel = kernels_of(T, k, d, f, S, I, dtype=dtype)[0]
    assert want is None or kernel == want
    R, rank = I // S, I // S - 1
    table = grace.GraceTable(I, R, 1, [0] * R, [1] * R, list(range(I + 1)), [e // S for e in range(I)])
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(T)
    x = torch.randn((T, d), generator=gen, device="cuda").to(tdt)
    wg, wu = ((0.05 * torch.randn((S, f, d), generator=gen, device="cuda")).to(tdt) for _ in range(2))
    share = torch.rand(I, generator=gen, device="cuda") ** 3
    ti = torch.multinomial(share, T * k, replacement=True, generator=gen).to(torch.int32).reshape(T, k)
    ti[T // 2, k - 1] = I + 3
    ti[0, 0] = -1
    pos, src, ioff, _, _, _ = grace.grace_permute(table, ti, None)
    n = int(ioff[-1])
    src[n:] = -7   # (positions of no row; whatever they hold, they are not the rank's)
    nbytes = grace.grace_workspace_bytes(T, I, k, I, d, f, 0, grace.GRACE_F32 if dtype == "f32" else grace.GRACE_BF16)
    results = []
    for one_call in (True, False):
        xp = torch.full((T * k, d), 3.0, dtype=tdt, device="cuda")
        ws, state = torch.zeros(nbytes, dtype=torch.uint8, device="cuda"), torch.zeros(8, dtype=torch.int32, device="cuda")
        if one_call:
            grace.grace_expert_ffn_up_share_scatter(table, rank, x, pos, src, xp, ioff, k, wg, wu, state, ws)
        else:
            grace.grace_permute_rows(x, pos, k, xp)
            grace.grace_expert_ffn_up_share(table, rank, xp, ioff, T, k, wg, wu, state, ws)
        results.append((xp, ws, state))
    for a, b in zip(*results):
        assert torch.equal(a, b)
    assert torch.equal(results[0][0][:n], x[(src[:n] // k).long()])


@pytest.mark.parametrize("T,k,d,f,S,I,want", [(2100, 17, 1024, 512, 20, 40, True), (100, 8, 2112, 1024, 32, 64, False), (1500, 64, 512, 512, 66, 66, True)])
def test_layer_has_its_rows_moved_where_the_projection_carries_them(T, k, d, f, S, I, want):
    """... and by the dispatch call elsewhere, also where the large tiles take the projection."""
    assert kernels_of(T, k, d, f, S, I)[0] == "persist"
    table = grace.GraceTable(I, I // S, 1, [0] * (I // S), [1] * (I // S), list(range(I + 1)), [e // S for e in range(I)])
    gen = torch.Generator(device="cuda").manual_seed(T)
    w = [(0.05 * torch.randn(s, generator=gen, device="cuda")).bfloat16() for s in ((S, f, d), (S, f, d), (S, d, f))]
    layer = grace.GraceMoELayer(table, 0, T, k, d, f, torch.bfloat16, *w)
    assert layer.gather_rows is want
    x, logits = torch.randn((T, d), generator=gen, device="cuda").bfloat16(), torch.randn((T, I), generator=gen, device="cuda")
    layer.forward(logits, x)
    assert torch.equal(layer.xp, x[(layer.perm_out[1] // k).long()])
    y = grace.grace_expert_ffn(table, 0, layer.xp, layer.perm_out[2], T, k, *w)
    assert torch.equal(layer.y, y)


@pytest.mark.parametrize("T,E,k,R,spread,policy,d,f,n_shared,dtype,kernel", [
    (1, 64, 8, 4, 2, 0, 2048, 1024, 0, "bf16", "stream"),       # one token, a wavefront for it
    (4, 64, 8, 4, 2, 1, 136, 200, 1, "bf16", "stream"),         # several candidates per expert; K of whole steps and 8 left over
    (5, 60, 4, 8, 2, 0, 256, 96, 3, "bf16", "stream"),          # four tokens per wavefront; experts that fill no 16 lanes
    (17, 33, 7, 4, 3, 1, 512, 352, 2, "bf16", "stream"),        # two fragments
    (64, 64, 8, 32, 1, 0, 512, 96, 0, "bf16", "stream"),        # four fragments, two experts per rank
    (16, 128, 8, 8, 2, 0, 2048, 768, 0, "bf16", "stream"),      # two experts per lane
    (32, 200, 5, 8, 1, 1, 256, 64, 0, "bf16", "stream"),        # four
    (9, 3, 3, 2, 2, 1, 64, 32, 2, "bf16", "stream"),            # every expert chosen; 16 tokens per look at the logits
    (40, 16, 2, 4, 2, 0, 128, 64, 1, "f32", "stream"),          # a lane per token
    (256, 8, 2, 4, 2, 0, 128, 256, 0, "f32", "stream"),         # pieces of 64 rows
    (255, 2, 1, 2, 1, 0, 64, 40, 0, "f32", "stream"),
    (16, 64, 8, 1, 1, 0, 4096, 200, 1, "bf16", "stream"),      # 64 slots of one rank, 16 columns per workgroup of the down projection
    (13, 10, 3, 2, 2, 1, 132, 68, 2, "f32", "stream"),         # last columns past the end, K of two steps and a rest
    (96, 64, 8, 2, 2, 1, 100, 36, 0, "f32", "stream"),          # all instances here and elsewhere
    (7, 40, 6, 4, 2, 1, 192, 600, 0, "bf16", "stream"),        # projection in units of 4 columns: a part of K of one step
    (8, 12, 9, 1, 1, 0, 64, 7400, 0, "bf16", "stream"),        # more than 64 units per workgroup
    (8, 12, 5, 2, 2, 1, 96, 516, 0, "f32", "stream"),
    (16, 12, 5, 2, 2, 1, 96, 516, 0, "f32", "stream"),
    (3, 200, 5, 8, 1, 1, 256, 64, 0, "f32", "stream"),
    (8, 100, 6, 8, 2, 0, 320, 520, 0, "bf16", "stream"),
    (64, 36, 8, 4, 1, 0, 512, 1408, 0, "bf16", "mid"),      # the 96-row kernel: four tokens per wavefront
    (95, 12, 7, 3, 3, 1, 264, 1480, 0, "bf16", "mid"),       # three words of tokens, several candidates
    (32, 100, 6, 16, 1, 1, 192, 2568, 0, "bf16", "mid"),     # eight experts per lane
    (96, 16, 2, 4, 1, 0, 320, 2096, 0, "bf16", "mid"),       # a lane per token
    (70, 16, 2, 16, 1, 0, 320, 2096, 0, "bf16", "mid"),      # tiles in halves
    (30, 140, 7, 16, 1, 1, 128, 1672, 0, "bf16", "mid"),     # a wavefront per token
])
def test_dispatch_joined_with_the_projection(T, E, k, R, spread, policy, d, f, n_shared, dtype, kernel):
    """The smallest batches' one launch for dispatch and gate+up projection gives what the separate calls give, and the rest of
    the step finds its rows (up to 16 tokens in one launch): ties, masked logits, carried counters, a second step whose rows move."""
    rng = np.random.default_rng(T + E)
    hosts = [sorted(rng.choice(R, size=rng.integers(1, spread + 1), replace=False).tolist()) for _ in range(E)]
    inst_ptr = np.concatenate([[0], np.cumsum([len(h) for h in hosts])]).astype(np.int32)
    table = grace.GraceTable(E, R, min(2, R), (np.arange(R) >= (R + 1) // 2).astype(np.int32) if R > 1 else [0],
                             rng.integers(1, 9, size=R).astype(np.uint32), inst_ptr, np.concatenate(hosts).astype(np.int32))
    rank = int(np.concatenate(hosts)[0])
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    dt = grace.GRACE_BF16 if dtype == "bf16" else grace.GRACE_F32
    assert grace.grace_dispatch_joins_ffn(table, rank, T, k, d, f, dt)
    assert grace.grace_ffn_kernel(True, T, d, f, dt, k=k, S=len(table.local_experts(rank)), I=table.I)[0] == kernel
    S = len(table.local_experts(rank))
    gen = torch.Generator(device="cuda").manual_seed(T)
    w = [(torch.randn(s, generator=gen, device="cuda") * 0.1).to(tdt) for s in ((S, f, d), (S, f, d), (S, d, f))]
    y, want_y = torch.zeros((T * k, d), dtype=tdt, device="cuda"), torch.zeros((T * k, d), dtype=tdt, device="cuda")
    state, want_state = (torch.zeros(8, dtype=torch.int32, device="cuda") for _ in range(2))
    ws, want_ws = (torch.empty(grace.grace_workspace_bytes(T, E, k, table.I, d, f, 0, dt), dtype=torch.uint8, device="cuda") for _ in range(2))
    ws2, want_ws2 = (torch.empty(grace.grace_workspace_bytes(T, 1, 1, 1, d, f, n_shared, dt), dtype=torch.uint8, device="cuda") for _ in range(2))
    sh = [(torch.randn((n_shared, *s), generator=gen, device="cuda") * 0.1).to(tdt) for s in ((f, d), (f, d), (d, f))] if n_shared else None
    ys, want_ys = (torch.zeros((T, d), dtype=tdt, device="cuda") if n_shared else None for _ in range(2))
    for step in range(2):
        logits = np.round(rng.standard_normal((T, E)) * 4).astype(np.float32) / 4
        logits[0, ::2] = -0.0
        logits[T // 2, 1:] = -np.inf
        rr = torch.from_numpy(rng.integers(0, 2 ** 32, size=E, dtype=np.uint64).astype(np.uint32).view(np.int32)).cuda()
        logits, x = torch.from_numpy(logits).cuda(), torch.randn((T, d), generator=gen, device="cuda").to(tdt)
        rr_out, want_rr = torch.empty_like(rr), torch.empty_like(rr)
        route, perm = grace.grace_dispatch_ffn_up_share(table, rank, logits, k, x, w[0], w[1], state, ws, rr_in=rr, rr_out=rr_out, policy=policy,
                                                        shared=sh and (sh[0], sh[1]), ws_shared=ws2)
        out = grace.grace_dispatch_ffn_down_share(table, rank, perm[2], perm[0], route[1], w[2], y, state, ws, sh and sh[2], ys, ws2)
        want_route = grace.grace_route(table, rank, logits, k, rr_in=rr, rr_out=want_rr, policy=policy)
        want_perm = grace.grace_permute(table, want_route[2], x)
        grace.grace_expert_ffn_up_share(table, rank, want_perm[5], want_perm[2], T, k, w[0], w[1], want_state, want_ws)
        grace.grace_expert_ffn_down_share(table, rank, want_perm[2], T, k, w[2], want_y, want_state, want_ws)
        if n_shared:
            grace.grace_shared_ffn_up(x, sh[0], sh[1], want_ws2)
            grace.grace_shared_ffn_down(sh[2], want_ws2, T, want_ys)
        torch.cuda.synchronize()
        for name, a, b in zip(("expert", "inst", "count", "pos", "src", "inst_off", "rank_off", "node_off", "xp", "state", "rr"),
                              (route[0], *route[2:], *perm, state, rr_out), (want_route[0], *want_route[2:], *want_perm, want_state, want_rr)):
            assert torch.equal(a, b), (step, name)
        torch.testing.assert_close(route[1], want_route[1], rtol=1e-6, atol=0)    # (sums of the exponentials in another order)
        # sums in another order: fp32 rounding of f products and, in bf16, the last bit of y and of what is made of it
        hosts_all = S == table.I
        want_out = grace.grace_combine(y, perm[0], route[1], ys) if hosts_all else grace.grace_combine_share(y, perm[0], route[1], state, ys)
        for name, a, b in (("y", y, want_y), ("y_shared", ys, want_ys), ("out", out, want_out)):
            if a is None:
                continue
            a, b = a.double(), b.double()
            assert torch.isfinite(a).all(), (step, name)
            assert (a == 0).equal(b == 0) or name == "y_shared" or dtype == "f32", (step, name)      # rows of others stay zero
            scale = b.abs().clamp(min=float(b.pow(2).mean().sqrt()))
            assert float(((a - b).abs() / scale).max()) <= (2.0 ** -7 if dtype == "bf16" else 1e-5), (step, name)


@pytest.mark.parametrize("T,E,k,R,n_shared,d,f", [
    (70, 8, 2, 2, 2, 72, 64),          # rows of nine 16-byte vectors, K segments of a step; few tiles, in halves
    (333, 16, 4, 4, 1, 512, 352),      # K of half a step past five
    (3001, 16, 3, 4, 2, 264, 72),      # many tokens for every mover; strips past N; K segments of 72
    (150, 140, 9, 2, 3, 136, 40),      # more than 64 slots
    (600, 8, 8, 8, 4, 128, 192),       # every token on every expert
    (90, 12, 4, 3, 0, 200, 72),        # no shared experts: projection and rows alone
    (2000, 32, 8, 4, 0, 128, 64),
])
def test_shared_and_expert_projections_in_one_launch(T, E, k, R, n_shared, d, f):
    """The joint launches give what the calls one after the other give, bit for bit, over two steps whose rows move."""
    rng = np.random.default_rng(T + E)
    table = grace.GraceTable(E, R, 1, [0] * R, [1] * R, list(range(E + 1)), [e * R // E for e in range(E)])
    rank, tdt = R - 1, torch.bfloat16
    S = len(table.local_experts(rank))
    sizes = dict(k=k, S=S, I=E)
    if n_shared:
        assert grace.grace_ffn_joins_shared(True, T, d, f, n_shared, **sizes) and grace.grace_ffn_joins_shared(False, T, d, f, n_shared, **sizes)
    else:
        assert grace.grace_ffn_kernel(True, T, d, f, **sizes)[0] == "mid" and grace.grace_ffn_joins_shared(True, T, d, f, 0, **sizes)
    gen = torch.Generator(device="cuda").manual_seed(T)
    normal = lambda *s: (torch.randn(s, generator=gen, device="cuda") * 0.1).to(tdt)
    w, sh = (normal(S, f, d), normal(S, f, d), normal(S, d, f)), (normal(n_shared, f, d), normal(n_shared, f, d), normal(n_shared, d, f))
    zeros = lambda *s: torch.zeros(s, dtype=tdt, device="cuda")
    state, want_state = (torch.zeros(8, dtype=torch.int32, device="cuda") for _ in range(2))
    ws, want_ws = (torch.empty(grace.grace_workspace_bytes(T, E, k, E, d, f), dtype=torch.uint8, device="cuda") for _ in range(2))
    ws2, want_ws2 = (torch.empty(grace.grace_workspace_bytes(T, 1, 1, 1, d, f, n_shared), dtype=torch.uint8, device="cuda") for _ in range(2))
    y, want_y, ys, want_ys = zeros(T * k, d), zeros(T * k, d), zeros(T, d), zeros(T, d)
    for step in range(2):
        logits = torch.from_numpy(rng.standard_normal((T, E)).astype(np.float32)).cuda()
        x = normal(T, d)
        route, (pos, src, ioff, roff, noff, _) = grace.grace_route_permute(table, rank, logits, k, None)
        xp, want_xp = (torch.full((T * k, d), 7.0, dtype=tdt, device="cuda") for _ in range(2))
        grace.grace_permute_rows(x, pos, k, want_xp)
        grace.grace_expert_ffn_up_share(table, rank, want_xp, ioff, T, k, w[0], w[1], want_state, want_ws)
        grace.grace_expert_ffn_down_share(table, rank, ioff, T, k, w[2], want_y, want_state, want_ws)
        if n_shared:
            grace.grace_shared_ffn_up(x, sh[0], sh[1], want_ws2)
            grace.grace_shared_ffn_down(sh[2], want_ws2, T, want_ys)
            grace.grace_expert_shared_ffn_up_scatter(table, rank, x, pos, src, xp, ioff, k, w[0], w[1], sh[0], sh[1], state, ws, ws2)
            grace.grace_expert_shared_ffn_down(table, rank, ioff, T, k, w[2], sh[2], y, ys, state, ws, ws2)
        else:
            grace.grace_expert_ffn_up_share_scatter(table, rank, x, pos, src, xp, ioff, k, w[0], w[1], state, ws)
            grace.grace_expert_ffn_down_share(table, rank, ioff, T, k, w[2], y, state, ws)
        torch.cuda.synchronize()
        for name, a, b in (("xp", xp, want_xp), ("y", y, want_y), ("y_shared", ys, want_ys), ("state", state, want_state)):
            assert torch.equal(a, b), (step, name)
        assert torch.isfinite(y.float()).all() and y.abs().max() > 0


def test_joined_step_in_the_workspace_of_a_larger_batch():
    """64 slots of one rank, rows by slots, in the buffer of 257 tokens: nothing behind it is written, and the calls without slots take it."""
    T, larger, E, k, d, f, bf = 64, 257, 64, 8, 256, 192, torch.bfloat16
    table = grace.GraceTable(E, 1, 1, [0], [1], list(range(E + 1)), [0] * E)
    assert grace.grace_dispatch_joins_ffn(table, 0, T, k, d, f)
    size = grace.grace_workspace_bytes(larger, E, k, E, d, f)
    held = torch.full((size + (4 << 20),), 0xA5, dtype=torch.uint8, device="cuda")
    ws = held[:size]
    gen = torch.Generator(device="cuda").manual_seed(1)
    logits, x = torch.randn((T, E), generator=gen, device="cuda"), torch.randn((T, d), generator=gen, device="cuda").to(bf)
    w = [(torch.randn(s, generator=gen, device="cuda") * 0.1).to(bf) for s in ((E, f, d), (E, f, d), (E, d, f))]
    y, state = torch.zeros((T * k, d), dtype=bf, device="cuda"), torch.zeros(8, dtype=torch.int32, device="cuda")
    route, perm = grace.grace_dispatch_ffn_up_share(table, 0, logits, k, x, w[0], w[1], state, ws)
    grace.grace_dispatch_ffn_down_share(table, 0, perm[2], perm[0], route[1], w[2], y, state, ws)
    want = grace.grace_expert_ffn(table, 0, perm[5], perm[2], T, k, *w, ws=ws)
    torch.cuda.synchronize()
    assert (held[size:] == 0xA5).all()
    assert float((y.double() - want.double()).abs().max()) <= 2.0 ** -7 * float(want.abs().max())


@pytest.mark.parametrize("T,k,d,f,S,n_shared,kernel", [(300, 4, 128, 64, 4, 0, "mid"), (300, 4, 128, 64, 4, 2, "mid"), (9000, 8, 512, 256, 8, 0, "persist")])
def test_stale_assignments_stay_inside_the_tokens(T, k, d, f, S, n_shared, kernel):
    """perm_src entries that are no assignment of the batch: read as some token's, the other rows are as without them."""
    I, bf = 2 * S, torch.bfloat16
    assert kernels_of(T, k, d, f, S, I)[0] == kernel
    table = grace.GraceTable(I, 2, 1, [0, 0], [1, 1], list(range(I + 1)), [e // S for e in range(I)])
    gen = torch.Generator(device="cuda").manual_seed(T)
    normal = lambda *s: (torch.randn(s, generator=gen, device="cuda") * 0.1).to(bf)
    x, w, sh = normal(T, d), (normal(S, f, d), normal(S, f, d)), (normal(n_shared, f, d), normal(n_shared, f, d))
    _, (pos, src, ioff, _, _, _) = grace.grace_route_permute(table, 0, torch.randn((T, I), generator=gen, device="cuda"), k, None)
    n = int(ioff[S])
    stale = src.clone()
    at = torch.arange(3, n, 7, device="cuda")
    stale[at] = torch.tensor([-1, -2 ** 31, 2 ** 31 - 1, T * k], dtype=torch.int32, device="cuda")[torch.arange(len(at), device="cuda") % 4]
    hidden = []
    for s in (src, stale):
        ws, state = torch.zeros(grace.grace_workspace_bytes(T, I, k, I, d, f), dtype=torch.uint8, device="cuda"), torch.zeros(8, dtype=torch.int32, device="cuda")
        xp = torch.zeros((T * k, d), dtype=bf, device="cuda")
        if n_shared:
            ws2 = torch.empty(grace.grace_workspace_bytes(T, 1, 1, 1, d, f, n_shared), dtype=torch.uint8, device="cuda")
            assert grace.grace_ffn_joins_shared(True, T, d, f, n_shared, k=k, S=S, I=I)
            grace.grace_expert_shared_ffn_up_scatter(table, 0, x, pos, s, xp, ioff, k, *w, *sh, state, ws, ws2)
        else:
            grace.grace_expert_ffn_up_share_scatter(table, 0, x, pos, s, xp, ioff, k, *w, state, ws)
        hidden.append(ws[:n * f * 2].view(bf).view(n, f))
    other = torch.ones(n, dtype=torch.bool, device="cuda")
    other[at] = False
    assert torch.equal(hidden[0][other], hidden[1][other]) and torch.isfinite(hidden[1].float()).all()


@pytest.mark.parametrize("T,E,k,d,f,dtype", [
    (2, 3, 3, 64, 64, "f32"),            # a wavefront per token, in units of columns
    (16, 6, 5, 64, 64, "f32"),           # a lane per token
    (40, 16, 15, 64, 32, "f32"),
    (13, 40, 20, 64, 32, "bf16"),        # four tokens per wavefront
    (12, 100, 60, 64, 16, "bf16"),       # experts in a lane: broadcast, and (k small) rounds
    (32, 70, 3, 64, 16, "bf16"),
    (96, 16, 2, 320, 2000, "bf16"),      # the 96-row kernel
])
def test_joined_dispatch_with_logits_that_are_no_numbers(T, E, k, d, f, dtype):
    """A token whose logits are NaN (any bits) or infinite spoils nothing but itself: tiles and dispatch see the same choices."""
    table = grace.GraceTable(E, 2, 1, [0, 0], [1, 1], list(range(E + 1)), [e % 2 for e in range(E)])
    tdt, dt = (torch.bfloat16, grace.GRACE_BF16) if dtype == "bf16" else (torch.float32, grace.GRACE_F32)
    assert grace.grace_dispatch_joins_ffn(table, 0, T, k, d, f, dt)
    S = len(table.local_experts(0))
    gen = torch.Generator(device="cuda").manual_seed(T)
    w = [(torch.randn(s, generator=gen, device="cuda") * 0.1).to(tdt) for s in ((S, f, d), (S, f, d), (S, d, f))]
    x, logits = torch.randn((T, d), generator=gen, device="cuda").to(tdt), torch.randn((T, E), generator=gen, device="cuda")
    bits = logits.view(torch.int32)
    odd = list(range(0, T, 3))
    for n, t in enumerate(odd):     # all ones, as few as leave it chosen or all; quiet NaN of either sign; infinities
        bits[t, (t + n) % E:] = [-1, 0x7FC00000, -1, 0x7F800000, -0x00400000][n % 5]
        if n % 2:
            bits[t, ::3] = [-1, -2, 0x7F800000][n % 3]
    y, state = torch.zeros((T * k, d), dtype=tdt, device="cuda"), torch.zeros(8, dtype=torch.int32, device="cuda")
    ws = torch.empty(grace.grace_workspace_bytes(T, E, k, E, d, f, 0, dt), dtype=torch.uint8, device="cuda")
    route, perm = grace.grace_dispatch_ffn_up_share(table, 0, logits, k, x, w[0], w[1], state, ws)
    out = grace.grace_dispatch_ffn_down_share(table, 0, perm[2], perm[0], route[1], w[2], y, state, ws)
    pos, ioff = perm[0].long().view(T, k), perm[2].long()
    assert ((pos >= 0) & (pos < T * k)).all() and pos.view(-1).unique().numel() == T * k        # every choice has its row
    assert torch.equal(perm[5][pos.view(-1)], x.repeat_interleave(k, 0))
    # in fp32: rows of this rank, and the tokens with ordinary logits
    want = torch.zeros((T * k, d), device="cuda")
    for s in range(S):
        r = slice(int(ioff[s]), int(ioff[s + 1]))
        a = perm[5][r].float()
        h = (torch.nn.functional.silu(a @ w[0][s].float().T) * (a @ w[1][s].float().T)).to(tdt).float()
        want[r] = h @ w[2][s].float().T
    plain = torch.tensor([t not in odd for t in range(T)], device="cuda")
    bound = 2.0 ** -6 if dtype == "bf16" else 1e-5      # two roundings of 2^-9 at most each, of values next to a rounding border the last digit
    assert float((y.float() - want).abs().max()) <= bound * float(want.abs().max())
    want_out = (want[pos] * route[1][..., None]).sum(1)
    assert torch.isfinite(out[plain].float()).all()
    assert float((out.float() - want_out)[plain].abs().max()) <= bound * float(want_out[plain].abs().max())


@pytest.mark.parametrize("T,k,d,n_shared", [(97, 3, 8, 2), (300, 4, 264, 0), (130, 2, 512, 1), (700, 5, 520, 2), (260, 64, 1032, 0), (3000, 2, 64, 1), (97, 3, 4104, 2)])
def test_rows_of_any_width_moved_beside_the_tiles(T, k, d, n_shared):
    """Pieces of a row: one of few lanes, whole ones, a last one of one lane; more pieces than wavefronts; positions outside the buffer."""
    S, E, f, bf = 2, 2 * k, 64, torch.bfloat16
    table = grace.GraceTable(E, 2, 1, [0, 0], [1, 1], list(range(E + 1)), [e >= S for e in range(E)])
    assert grace.grace_ffn_joins_shared(True, T, d, f, n_shared, k=k, S=S, I=E)
    gen = torch.Generator(device="cuda").manual_seed(T)
    normal = lambda *s: (torch.randn(s, generator=gen, device="cuda") * 0.1).to(bf)
    x, w, sh = normal(T, d), (normal(S, f, d), normal(S, f, d)), (normal(n_shared, f, d), normal(n_shared, f, d))
    _, (pos, src, ioff, _, _, _) = grace.grace_route_permute(table, 0, torch.randn((T, E), generator=gen, device="cuda"), k, None)
    dropped = pos.clone()
    dropped[::11], dropped[5::13] = -1, T * k
    xp, want = (torch.full((T * k + 4, d), 7.0, dtype=bf, device="cuda") for _ in range(2))
    grace.grace_permute_rows(x, dropped, k, want)
    ws, state = torch.empty(grace.grace_workspace_bytes(T, E, k, E, d, f), dtype=torch.uint8, device="cuda"), torch.zeros(8, dtype=torch.int32, device="cuda")
    if n_shared:
        ws2 = torch.empty(grace.grace_workspace_bytes(T, 1, 1, 1, d, f, n_shared), dtype=torch.uint8, device="cuda")
        grace.grace_expert_shared_ffn_up_scatter(table, 0, x, dropped, src, xp, ioff, k, *w, *sh, state, ws, ws2)
    else:
        grace.grace_expert_ffn_up_share_scatter(table, 0, x, dropped, src, xp, ioff, k, *w, state, ws)
    assert torch.equal(xp, want)


@pytest.mark.parametrize("d,n_shared", [(256, 0), (512, 0), (256, 2), (512, 2)])
def test_narrow_rows_do_not_hold_up_the_launch_that_moves_them(d, n_shared):
    """A step with the rows moved beside the tiles against one with a launch for them: no slower.  (Twice as slow when a workgroup took a token at a
    time; the bound leaves room for noise.)"""
    T, k, E, f, bf = 1000, 2, 16, 352, torch.bfloat16
    table = grace.GraceTable(E, 4, 1, [0] * 4, [1] * 4, list(range(E + 1)), [e // 4 for e in range(E)])
    gen = torch.Generator(device="cuda").manual_seed(d)
    normal = lambda *s: (torch.randn(s, generator=gen, device="cuda") * 0.1).to(bf)
    shared = (normal(n_shared, f, d), normal(n_shared, f, d), normal(n_shared, d, f)) if n_shared else None
    layer = grace.GraceMoELayer(table, 0, T, k, d, f, bf, normal(4, f, d), normal(4, f, d), normal(4, d, f), shared=shared)
    logits, x = torch.randn((T, E), generator=gen, device="cuda"), normal(T, d)
    assert layer.join_shared[True] if n_shared else layer.gather_rows
    times = []
    for joint in (True, False):
        if not joint:
            layer.gather_rows, layer.join_shared, layer._key = False, [False, False], None
        layer.forward(logits, x)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(10):
                layer.forward(logits, x)
        layer._key = None
        best = float("inf")
        for _ in range(10):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record(); graph.replay(); b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        times.append(best)
    assert times[0] <= 1.3 * times[1], times


@pytest.mark.parametrize("T,k,R,n_shared,d,f,dtype", [
    (16, 5, 3, 0, 256, 64, "bf16"), (5, 3, 3, 2, 512, 96, "bf16"), (8, 7, 2, 1, 132, 68, "f32"), (16, 5, 1, 1, 256, 64, "f32"), (3, 3, 1, 0, 2048, 64, "bf16"),
])
def test_joined_combine_of_weights_that_are_no_numbers(T, k, R, n_shared, d, f, dtype):
    """Gate weights that are not finite, of this rank's rows and of others', and dropped positions: the one launch for the down projections and the
    combine makes of its y what the combine makes of it, bit for bit."""
    E, (tdt, dt) = 9, (torch.bfloat16, grace.GRACE_BF16) if dtype == "bf16" else (torch.float32, grace.GRACE_F32)
    table = grace.GraceTable(E, R, 1, [0] * R, [1] * R, list(range(E + 1)), [e % R for e in range(E)])
    assert grace.grace_dispatch_joins_ffn(table, 0, T, k, d, f, dt, n_shared=n_shared) == 2
    S = len(table.local_experts(0))
    gen = torch.Generator(device="cuda").manual_seed(T)
    normal = lambda *s: (torch.randn(s, generator=gen, device="cuda") * 0.1).to(tdt)
    w, sh = [normal(S, f, d), normal(S, f, d), normal(S, d, f)], [normal(n_shared, f, d), normal(n_shared, f, d), normal(n_shared, d, f)] if n_shared else None
    y, ys, state = normal(T * k, d).zero_(), normal(T, d) if n_shared else None, torch.zeros(8, dtype=torch.int32, device="cuda")
    ws = torch.empty(grace.grace_workspace_bytes(T, E, k, E, d, f, 0, dt), dtype=torch.uint8, device="cuda")
    ws2 = torch.empty(grace.grace_workspace_bytes(T, 1, 1, 1, d, f, n_shared, dt), dtype=torch.uint8, device="cuda")
    route, perm = grace.grace_dispatch_ffn_up_share(table, 0, torch.randn((T, E), generator=gen, device="cuda"), k, normal(T, d), w[0], w[1], state, ws,
                                                    shared=sh and sh[:2], ws_shared=ws2)
    pos, weight = perm[0].view(T, k).clone(), route[1].clone()
    here = pos < int(perm[2][S])     # (rank 0's rows are the first ones)
    spoilt = torch.zeros(T, dtype=torch.bool, device="cuda")
    for n, t in enumerate(range(0, T, 2)):
        of = torch.nonzero(here[t] if n % 3 == 0 or R == 1 else ~here[t]).view(-1).tolist()
        if not of:
            continue
        weight[t, of[-1]] = [float("nan"), float("inf"), -float("inf")][n % 3]
        if n % 4 == 3:
            pos[t, of[-1]] = T * k   # no row at all: its weight does not matter
        else:
            spoilt[t] = True
    pos[1::4, 0] = -1
    out = grace.grace_dispatch_ffn_down_share(table, 0, perm[2], pos.view(-1), weight, w[2], y, state, ws, sh and sh[2], ys, ws2)
    want = grace.grace_combine(y, pos.view(-1), weight, ys) if R == 1 else grace.grace_combine_share(y, pos.view(-1), weight, state, ys)
    torch.cuda.synchronize()
    assert spoilt.any() and torch.equal(torch.isfinite(out.float()).all(1), ~spoilt)
    assert torch.equal(out.isnan(), want.isnan()) and torch.equal(out.nan_to_num(), want.nan_to_num())
