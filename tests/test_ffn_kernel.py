"""Which kernel the FFN projections take, and the launches' sizes: host arithmetic, no GPU."""
import pytest

import paper_2509_25041_amd as grace

N_CU = 256
F32, BF16 = grace.GRACE_F32, grace.GRACE_BF16


@pytest.mark.parametrize("up,T,k,d,f,n_shared,S,I,dt", [
    (True, 150000, 8, 1024, 14336, 0, 8, 64, F32),        # hidden activation of 69 GB: 16 columns and 64 rows per workgroup are too many workgroups
    (True, 1200000, 1, 256, 14336, 1, 1, 1, F32),
    (True, 150000, 8, 200, 90000, 0, 8, 64, BF16),        # K no multiple of 64, hidden activation of 216 GB
    (True, 8, 1, 8, 2 ** 26, 0, 8, 8, BF16),              # decode batch, 2^26 columns of 16 bytes
    (False, 1000000, 2, 36864, 104, 0, 8, 64, BF16),
    (True, 32768, 6, 2048, 1408, 2, 1, 1, BF16),          # ordinary ones
    (False, 1, 8, 2048, 1024, 0, 18, 72, BF16),
    (True, 1000, 2, 1024, 2816, 0, 8, 16, F32),
    (True, 96 * 5592403, 1, 72, 192, 1, 1, 1, BF16),      # 2^24 - 7 tiles: 2^32 work-items once they are rounded up to whole runs
    (True, 96 * 5592403, 1, 72, 192, 0, 1, 1, BF16),
    (True, 96 * 5592403, 1, 64, 96, 1, 1, 1, F32),
    (False, 96 * 5592403, 1, 384, 72, 0, 1, 1, BF16),
])
def test_launch_fits_32_bits_of_work_items(up, T, k, d, f, n_shared, S, I, dt):
    """HIP refuses a launch of 2^32 work-items or more along one axis."""
    kernel, items = grace.grace_ffn_kernel(up, T, d, f, dt, k=k, S=S, I=I, n_shared=n_shared, n_cu=N_CU)
    assert 0 < items < 2 ** 32, (kernel, items)


@pytest.mark.parametrize("tiles", [1, 64, 192, 256, 257, 352, 384, 385, 396, 432, 448, 511, 512])
def test_tiles_of_the_shared_experts_run_all_at_once(tiles):
    """Up to two 96-row tiles per compute unit: whole or in part halved, not more workgroups than the units take at a time."""
    kernel, items = grace.grace_ffn_kernel(True, 96 * tiles - 5, 72, 64, BF16, n_shared=1, n_cu=N_CU)
    assert kernel == "mid" and tiles * 256 <= items <= 2 * N_CU * 256


def test_invalid_arguments_are_refused():
    for bad in (dict(T=0), dict(k=0), dict(S=0), dict(S=3, I=2), dict(d=12), dict(n_shared=-1), dict(n_cu=-1)):
        a = {**dict(T=4, d=64, f=64, k=1, S=1, I=1, n_shared=0, n_cu=N_CU), **bad}
        with pytest.raises(grace.GraceError):
            grace.grace_ffn_kernel(True, a["T"], a["d"], a["f"], BF16, k=a["k"], S=a["S"], I=a["I"], n_shared=a["n_shared"], n_cu=a["n_cu"])
    assert grace.load_library().grace_ffn_kernel(1, 4, 1, 64, 64, 0, 1, 1, BF16, N_CU, None, None) == -1


# (up, T, k, d, f, S, I): projections of one rank (S of I instances).  us on the 96-row kernel / on 256 x 256 tiles, with cold weights and the
# rank's even share of the rows in Zipf-shaped segments; where the host does not know the rows the choice looks at higher loads too.
@pytest.mark.parametrize("up,T,k,d,f,S,I,want", [
    (True, 3583, 4, 2048, 1408, 7, 64, "persist"),      # 37.9 / 47.4, at 7/4 of the share the large tiles still take one round
    (True, 2756, 8, 2048, 768, 19, 134, "persist"),     # 41.6 / 48.6, likewise
    (True, 1630, 2, 4096, 1792, 8, 8, "persist"),       # 161.6 / 96.3: every instance here
    (True, 1630, 2, 4096, 3584, 8, 8, "persist"),       # 289.8 / 189.4
    (True, 2120, 8, 2048, 256, 64, 64, "persist"),      # 73.5 / 51.0
    (False, 1254, 8, 2048, 768, 19, 134, "persist"),    # 22.3 / 22.3
    (False, 64, 4, 2048, 1408, 60, 60, "mid"),          # 45.4 / 57.4; streaming 48.7
    (False, 48, 6, 2048, 1408, 64, 64, "mid"),          # 46.6 / 57.5; streaming 52.6
])
def test_large_tiles_where_they_are_faster(up, T, k, d, f, S, I, want):
    assert grace.grace_ffn_kernel(up, T, d, f, BF16, k=k, S=S, I=I, n_cu=N_CU)[0] == want


@pytest.mark.parametrize("T,d,f,n_shared", [(2756, 2048, 704, 2), (6055, 2048, 704, 2), (1254, 2048, 1408, 2), (571, 2048, 1408, 4)])
def test_shared_projection_keeps_the_row_scatter(T, d, f, n_shared):
    """Gate+up projections of shared experts that are slower without the large-tile kernel, which carries the row scatter
    (65.8 / 58.4, 128.7 / 113.4, 56.3 / 53.2 and 54.6 / 45.5 us, the scatter of six or four rows per token included)."""
    assert grace.grace_ffn_kernel(True, T, d, f, BF16, n_shared=n_shared, n_cu=N_CU)[0] == "persist"


@pytest.mark.parametrize("up,T,k,d,f,n_shared,S,I,want", [
    (True, 1, 8, 2048, 1024, 0, 16, 66, "stream"), (False, 64, 8, 2048, 1024, 0, 16, 66, "stream"),
    (True, 64, 8, 2048, 1024, 0, 16, 66, "mid"), (True, 200, 8, 2048, 1024, 0, 16, 66, "mid"),
    (True, 500, 8, 2048, 768, 0, 16, 130, "mid"), (False, 2000, 2, 4096, 3584, 0, 1, 10, "mid"),
    (True, 200, 8, 2048, 1024, 0, 64, 64, "mid"), (True, 300, 1, 2048, 1408, 2, 1, 1, "mid"),
    (True, 32768, 1, 2048, 1408, 2, 1, 1, "persist"), (True, 8192, 8, 2048, 768, 0, 16, 130, "persist"),
    (False, 3001, 6, 2048, 352, 0, 2, 69, "mid"),       # K no multiple of 64
    (False, 21, 8, 2048, 384, 0, 128, 128, "stream"),   # 11.4 us, 14.2 with the 96-row kernel
    (False, 33, 8, 2048, 384, 0, 128, 128, "mid"), (False, 16, 8, 2048, 1408, 0, 64, 64, "stream"),
])
def test_kernels_over_the_batch_sizes(up, T, k, d, f, n_shared, S, I, want):
    assert grace.grace_ffn_kernel(up, T, d, f, BF16, k=k, S=S, I=I, n_shared=n_shared, n_cu=N_CU)[0] == want


@pytest.mark.parametrize("up,T,k,d,f,n_shared,S,I,want", [
    # streaming kernel / split kernel ("mid"), us
    (True, 2000, 8, 2048, 768, 0, 4, 8, "mid"),          # 493 / 238
    (False, 2000, 8, 2048, 768, 0, 4, 8, "mid"),         # 241 / 140
    (False, 5000, 1, 2048, 768, 1, 1, 1, "mid"),         # 179 / 96
    (True, 500, 8, 1024, 2816, 0, 16, 64, "mid"),        # 231 / 136
    (False, 500, 8, 1024, 2816, 0, 16, 64, "mid"),       # 127 / 78
    (True, 500, 2, 548, 2816, 0, 8, 16, "mid"),          # 69 / 41
    (True, 300, 8, 1024, 1388, 0, 16, 16, "mid"),        # 156 / 91
    (True, 65, 2, 1024, 1388, 0, 16, 64, "stream"),      # 33 / 28: two rows per segment are expected, there may be fewer
    (False, 1000, 8, 2048, 768, 0, 16, 16, "mid"),       # 236 / 140
    (False, 128, 8, 2048, 768, 0, 16, 16, "mid"),        # 53 / 43
    (True, 200, 8, 2048, 768, 0, 4, 8, "mid"),           # 72 / 48
    (True, 500, 2, 548, 1388, 0, 16, 16, "mid"),         # 65 / 41
    (True, 1000, 1, 2048, 768, 1, 1, 1, "mid"),          # 68 / 57
    (False, 1000, 1, 2048, 2048, 2, 1, 1, "mid"),        # 172 / 127
    (False, 100, 2, 1024, 2816, 0, 9, 18, "mid"),        # 56 / 35: groups that share K
    (False, 2000, 2, 1024, 1388, 0, 9, 18, "mid"),       # 60 / 45
    (True, 130, 1, 2048, 768, 1, 1, 1, "stream"),        # 23 / 35: few tiles
    (False, 130, 1, 2048, 768, 1, 1, 1, "stream"),       # 11.4 / 13.6
    (True, 70, 1, 2048, 352, 0, 1, 4, "stream"),         # 14.3 / 27.8
    (True, 338, 1, 512, 1024, 0, 2, 4, "stream"),        # 15.6 / 13.2
    (True, 74, 1, 1024, 512, 0, 64, 128, "stream"),      # 20.2 / 22.0: fewer rows than segments
    (False, 300, 8, 768, 256, 0, 16, 16, "stream"),      # 18.7 / 16.7: short K, about a tile per unit
    (False, 65, 1, 1024, 1388, 2, 1, 1, "mid"),          # vector ALUs 329 / 34: K segments of 1388 are not for the streaming kernel
    (False, 64, 1, 1024, 1388, 2, 1, 1, "vector_f32"),
    (False, 90, 1, 515, 200, 3, 1, 1, "mid"),            # output rows that are no whole vectors
    (True, 64, 2, 1024, 2816, 0, 16, 16, "stream"), (False, 64, 2, 1024, 2816, 0, 16, 16, "stream"),    # up to 64 tokens
])
def test_f32_kernels_over_the_batch_sizes(up, T, k, d, f, n_shared, S, I, want):
    assert grace.grace_ffn_kernel(up, T, d, f, F32, k=k, S=S, I=I, n_shared=n_shared, n_cu=N_CU)[0] == want


@pytest.mark.parametrize("T,k,d,f,n_shared,S,I,dt,want", [
    (7001, 8, 2048, 768, 0, 16, 130, BF16, True), (32768, 6, 2048, 1408, 2, 1, 1, BF16, True),
    (100, 8, 2112, 1024, 0, 32, 64, BF16, False),        # large tiles, rows that are no whole 1 KB
    (2000, 65, 2048, 1024, 0, 66, 66, BF16, False),      # more choices than a wavefront has lanes
    (1500, 65, 512, 1024, 2, 1, 1, BF16, False), (1500, 64, 512, 1024, 2, 1, 1, BF16, True),
    (524288, 2, 2048, 1024, 0, 8, 8, BF16, False),       # tokens of 2 GB: the experts' kernel reads them at 32-bit offsets ...
    (524288, 2, 2048, 1024, 1, 1, 1, BF16, True),        # ... the shared experts' moves rows at 64-bit ones
    (2 ** 28, 2, 512, 1024, 1, 1, 1, BF16, False),       # T * k of 2^29
    (200, 8, 2048, 1024, 0, 16, 66, BF16, False), (5000, 8, 2048, 768, 0, 4, 8, F32, False),   # other kernels
])
def test_rows_carried_by_the_gate_up_projection(T, k, d, f, n_shared, S, I, dt, want):
    kernel = grace.grace_ffn_kernel(True, T, d, f, dt, k=k, S=S, I=I, n_shared=n_shared, n_cu=N_CU)[0]
    assert grace.grace_ffn_carries_rows(T, d, f, dt, k=k, S=S, I=I, n_shared=n_shared, n_cu=N_CU) == want
    assert kernel == ("persist" if S != 16 or I != 66 else "mid") or dt == F32


def test_row_query_refuses_what_the_kernel_query_refuses():
    for bad in (dict(T=0), dict(k=0), dict(d=12, f=8), dict(S=3, I=2)):
        a = {**dict(T=4, d=64, f=64, k=1, S=1, I=1), **bad}
        with pytest.raises(grace.GraceError):
            grace.grace_ffn_carries_rows(a["T"], a["d"], a["f"], BF16, k=a["k"], S=a["S"], I=a["I"], n_cu=N_CU)
    assert grace.load_library().grace_ffn_carries_rows(4, 1, 64, 64, 0, 1, 1, BF16, N_CU, None) == -1


@pytest.mark.parametrize("up,T,k,d,f,n_shared,S,I,dt,want", [
    (True, 3001, 6, 2048, 352, 2, 2, 69, BF16, True), (False, 3001, 6, 2048, 352, 2, 2, 69, BF16, True),
    (True, 32768, 6, 2048, 1408, 2, 3, 69, BF16, False),      # large tiles
    (True, 16, 6, 2048, 1408, 2, 3, 69, BF16, False),         # streamed
    (True, 200, 4, 2048, 1408, 2, 0, 69, BF16, False),        # no instance here
    (True, 1000, 4, 1024, 1024, 1, 4, 8, F32, False),
    (True, 512, 8, 2048, 1024, 0, 16, 66, BF16, True), (False, 512, 8, 2048, 1024, 0, 16, 66, BF16, False),   # the rows: gate+up alone
    (True, 200, 2, 4096, 3584, 0, 1, 10, BF16, False), (True, 512, 2, 4096, 3584, 0, 1, 10, BF16, True),
])
def test_projections_joined_with_the_shared_experts(up, T, k, d, f, n_shared, S, I, dt, want):
    assert grace.grace_ffn_joins_shared(up, T, d, f, n_shared, dt, k=k, S=S, I=I, n_cu=N_CU) == want
