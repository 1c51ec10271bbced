"""Offsets of the weight loads along a K axis in segments, checked on the host against 64-bit arithmetic."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_25041_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "kseg_walk.h"
// args: K segments, their length, elements between them.  Walks all lanes' chunks of 8 elements in steps of 64, eight steps
// further than K, as the kernel's look-ahead does; prints the number of wrong offsets.
int main(int, char **v) {
    const int n = atoi(v[1]), len = atoi(v[2]), K = n * len;
    const long long stride = atoll(v[3]);
    long long wrong = 0;
    for (int chunk = 0; chunk < 8; ++chunk) {
        grace::KSegWalk walk{chunk * 8};
        for (int k0 = 0; k0 < (K + 63) / 64 * 64 + 8 * 64; k0 += 64) {
            const int k = k0 + chunk * 8;
            const uint32_t add = walk.next(k, K, len, stride, 64);
            const uint32_t row = 31u * (uint32_t)len * 2u, got = grace::offset_with(row, add);
            const long long want = row + ((long long)(k / len) * (stride - len)) * 2;
            wrong += k < K ? got != want : got < grace::NO_DATA;
            wrong += grace::offset_with(grace::NO_DATA, add) < grace::NO_DATA;
        }
    }
    printf("%lld\n", wrong);
}
"""


@pytest.mark.parametrize("n_seg,seg_len,stride", [
    (2, 1408, 2048 * 1408), (3, 40, 520 * 40), (2, 8, 64), (4, 352, 2048 * 352),
    (3, 4096, 123456 * 4096),            # 3 GB of weights: the last segment starts below 2 GiB, its end lies beyond
    (2, 32768, 32760 * 32768),           # 4 GB
    (129, 8, 1048568 * 8),               # many short segments: the look-ahead passes 64 further ones
])
def test_offsets_along_k_segments(tmp_path, n_seg, seg_len, stride):
    assert (n_seg - 1) * stride * 2 < 2 ** 31       # what the launcher lets through
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe), str(n_seg), str(seg_len), str(stride)], check=True, capture_output=True, text=True)
    assert int(out.stdout) == 0
