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
])
def test_launch_fits_32_bits_of_work_items(up, T, k, d, f, n_shared, S, I, dt):
    """HIP refuses a launch of 2^32 work-items or more along one axis."""
    kernel, items = grace.grace_ffn_kernel(up, T, d, f, dt, k=k, S=S, I=I, n_shared=n_shared, n_cu=N_CU)
    assert 0 < items < 2 ** 32, (kernel, items)


def test_invalid_arguments_are_refused():
    for bad in (dict(T=0), dict(k=0), dict(S=0), dict(S=3, I=2), dict(d=12), dict(n_shared=-1), dict(n_cu=-1)):
        a = {**dict(T=4, d=64, f=64, k=1, S=1, I=1, n_shared=0, n_cu=N_CU), **bad}
        with pytest.raises(grace.GraceError):
            grace.grace_ffn_kernel(True, a["T"], a["d"], a["f"], BF16, k=a["k"], S=a["S"], I=a["I"], n_shared=a["n_shared"], n_cu=a["n_cu"])
    assert grace.load_library().grace_ffn_kernel(1, 4, 1, 64, 64, 0, 1, 1, BF16, N_CU, None, None) == -1
