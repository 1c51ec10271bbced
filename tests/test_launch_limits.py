"""Launches of the library's calls against what HIP takes, on the host: a recorder stands in for the runtime."""
import os
import subprocess
import sys

import pytest

import paper_2509_25041_amd as grace
from paper_2509_25041_amd.layer import dispatch_is_one_launch

HERE = os.path.dirname(os.path.abspath(__file__))

PRELUDE = r"""
import ctypes as C
import sys
recorder = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)   # ahead of the runtime that the library is linked with
lib = C.CDLL(sys.argv[2])
i32, at = C.c_int32, C.c_void_p(1 << 20)             # (no kernel runs: nothing is behind the device addresses)
lib.grace_last_error.restype = C.c_char_p

def table(E, R):
    h, ints = C.c_void_p(), lambda v: (i32 * len(v))(*v)
    rc = lib.grace_table_create(C.byref(h), E, R, 1, ints([0] * R), ints([1] * R), ints(list(range(E + 1))), ints([e * R // E for e in range(E)]), None)
    assert rc == 0, lib.grace_last_error()
    return h
"""

PROGRAM = PRELUDE + r"""
count = n_joined = wide = 0
for E, R, k in ((64, 32, 8), (64, 4, 8), (64, 1, 8), (8, 4, 2), (8, 1, 2), (128, 16, 8), (200, 100, 4), (16, 16, 1), (3, 3, 2)):
    h = table(E, R)
    for T in (1, 4, 7, 8, 9, 16, 17, 32, 33, 64, 65, 96, 97, 256, 512):
        for d, f in ((512, 96), (2048, 1024), (4096, 32), (1024, 352), (128, 256), (3072, 24)):
            for dt, shared in ((0, 0), (1, 0), (0, 2), (1, 2)):
                joined = i32()
                assert lib.grace_dispatch_joins_ffn(h, 0, T, k, d, f, shared, dt, 256, C.byref(joined)) == 0
                sh = at if shared else None
                before = C.c_int.in_dll(recorder, "n_recorded").value
                rc = lib.grace_dispatch_ffn_up_share(h, 0, 0, at, T, E, k, 1, None, None, at, at, at, at, at, d, f, shared, dt, at, at, at, at, at, at,
                                                     at, at, sh, sh, at, at, sh, None)
                assert rc == 0, lib.grace_last_error()
                rc = lib.grace_dispatch_ffn_down_share(h, 0, at, at, at, T, k, d, f, shared, dt, at, sh, at, sh, at, at, sh, at, None)
                assert rc == 0, lib.grace_last_error()
                launches = C.c_int.in_dll(recorder, "n_recorded").value - before
                assert launches >= 2
                assert recorder.launches_refused() == 0, (E, R, k, T, d, f, dt, shared, joined.value)
                count, n_joined, wide = count + launches, n_joined + (joined.value > 0), wide + (joined.value > 0 and 16 < T <= 64)
                C.c_int.in_dll(recorder, "n_recorded").value = 0
print(count, n_joined, wide)
"""


def run(tmp_path, program, *args):
    grace.load_library()   # (built if it is not)
    recorder = tmp_path / "recorder.so"
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", os.path.join(HERE, "launch_recorder.c"), "-o", str(recorder)], check=True)
    done = subprocess.run([sys.executable, "-c", program, str(recorder), grace.library_path(), *args], capture_output=True, text=True)
    assert done.returncode == 0, done.stderr[-2000:]
    return done.stdout


def test_launches_of_a_step_are_ones_that_hip_takes(tmp_path):
    """Dynamic LDS past 64 KB has to be allowed for the kernel first; work-items along x fit 32 bits."""
    count, joined, wide = map(int, run(tmp_path, PROGRAM).split())
    assert count > 2000 and joined > 500 and wide > 100


RULE = PRELUDE + r"""
class Launch(C.Structure):
    _fields_ = [("kernel", C.c_void_p), ("groups", C.c_uint32), ("threads", C.c_uint32), ("lds", C.c_uint64)]
E, R, T, k, d, f, shared, dt = map(int, sys.argv[3].split())
h, joined, sh = table(E, R), i32(), at if shared else None
assert lib.grace_dispatch_joins_ffn(h, 0, T, k, d, f, shared, dt, 256, C.byref(joined)) == 0
assert lib.grace_dispatch_ffn_up_share(h, 0, 0, at, T, E, k, 1, None, None, at, at, at, at, at, d, f, shared, dt, at, at, at, at, at, at, at, at, sh, sh, at,
                                       at, sh, None) == 0, lib.grace_last_error()
print(joined.value, C.c_int.in_dll(recorder, "n_recorded").value, Launch.in_dll(recorder, "recorded").threads // 64)
"""
F32, BF16 = grace.GRACE_F32, grace.GRACE_BF16


@pytest.mark.parametrize("E,R,T,k,d,f,shared,dt,joined,waves", [
    # many workgroups of slots without rows (the first one 74 us in two launches, 118 in one)
    (128, 1, 15, 2, 512, 3584, 0, BF16, 0, None), (64, 2, 22, 2, 512, 2816, 0, BF16, 0, None), (64, 1, 9, 4, 512, 2048, 0, BF16, 0, None),
    (128, 1, 8, 2, 512, 2048, 1, BF16, 0, None), (64, 1, 4, 6, 512, 2048, 1, F32, 0, None), (64, 4, 15, 8, 2048, 1024, 0, BF16, 2, 4),
    (128, 2, 16, 4, 1024, 512, 0, BF16, 1, 4), (16, 1, 14, 6, 1536, 2048, 0, F32, 0, None), (128, 1, 2, 4, 256, 3584, 0, BF16, 1, 8),
    # pieces of 64 rows: resident at once or not (the first one 34 and 51 us)
    (60, 16, 195, 2, 1024, 352, 0, F32, 0, None), (64, 16, 104, 1, 512, 1024, 0, F32, 0, None), (64, 16, 79, 6, 512, 352, 0, F32, 1, 8),
    (8, 4, 256, 2, 128, 256, 0, F32, 1, 4), (16, 8, 219, 1, 1536, 704, 0, F32, 0, None), (16, 8, 219, 1, 1536, 512, 0, F32, 1, 4),
    # narrow rows, many choices of many experts (the first one 18 us, 22 in one launch of 4 wavefronts, 16 of 16)
    (128, 16, 30, 8, 64, 352, 0, BF16, 1, 16), (64, 8, 63, 8, 256, 512, 0, BF16, 1, 8), (128, 8, 30, 6, 128, 704, 0, BF16, 0, None),
    (128, 8, 16, 8, 2048, 768, 0, BF16, 2, 4),
    # the 96-row kernel's tiles beside a dispatch that is longer than they are
    (64, 16, 89, 8, 256, 3584, 0, BF16, 0, None), (64, 16, 89, 8, 512, 3584, 0, BF16, 1, 4),
])
def test_smallest_batches_are_joined_where_that_is_faster(tmp_path, E, R, T, k, d, f, shared, dt, joined, waves):
    """One launch for dispatch and gate+up projection by the number of its workgroups and what they repeat; the query and the call agree."""
    said, launches, first = map(int, run(tmp_path, RULE, f"{E} {R} {T} {k} {d} {f} {shared} {dt}").split())
    assert said == joined
    assert (launches == 1) == (said > 0)
    if waves:
        assert first == waves


DISPATCH = PRELUDE + r"""
for E in (3, 64, 65, 200):
    for k in (1, 2, 3, 11):
        for T in (1, 32, 33, 85, 94, 96, 97, 256, 257) if k <= E else ():
            for I in (E, 300):
                h, ints = C.c_void_p(), lambda v: (i32 * len(v))(*v)
                n = [I - E + 1] + [1] * (E - 1)
                R = max(n)
                assert lib.grace_table_create(C.byref(h), E, R, 1, ints([0] * R), ints([1] * R), ints([sum(n[:e]) for e in range(E + 1)]), ints(list(range(n[0])) + [0] * (E - 1)),
                                              None) == 0, lib.grace_last_error()
                C.c_int.in_dll(recorder, "n_recorded").value = 0
                assert lib.grace_route_permute(h, 0, 0, at, T, E, k, 1, None, None, at, at, at, at, at, 64, 1, at, at, at, at, at, at, at, None) == 0, lib.grace_last_error()
                print(T, k, E, I, C.c_int.in_dll(recorder, "n_recorded").value)
                lib.grace_table_destroy(h)
"""


def test_layer_knows_where_the_dispatch_is_one_launch(tmp_path):
    """The layer leaves the rows to such a dispatch, whose launch is no shorter without them."""
    lines = [tuple(map(int, line.split())) for line in run(tmp_path, DISPATCH).splitlines()]
    assert len(lines) > 200 and {n == 1 for *_, n in lines} == {True, False}
    for *sizes, launches in lines:
        assert dispatch_is_one_launch(*sizes) == (launches == 1), (sizes, launches)
