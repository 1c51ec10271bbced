"""Launches of the library's calls against what HIP takes, on the host: a recorder stands in for the runtime."""
import os
import subprocess
import sys

import pytest

import paper_2509_25041_amd as grace

HERE = os.path.dirname(os.path.abspath(__file__))

PROGRAM = r"""
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


def test_launches_of_a_step_are_ones_that_hip_takes(tmp_path):
    """Dynamic LDS past 64 KB has to be allowed for the kernel first; work-items along x fit 32 bits."""
    grace.load_library()   # (built if it is not)
    recorder = tmp_path / "recorder.so"
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", os.path.join(HERE, "launch_recorder.c"), "-o", str(recorder)], check=True)
    run = subprocess.run([sys.executable, "-c", PROGRAM, str(recorder), grace.library_path()], capture_output=True, text=True)
    assert run.returncode == 0, run.stderr[-2000:]
    count, joined, wide = map(int, run.stdout.split())
    assert count > 2000 and joined > 500 and wide > 100
