"""Offsets of the weight loads along a K axis in segments, checked on the host against 64-bit arithmetic."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_25041_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "kseg_walk.h"
// args: K segments, their length, elements between them, bytes per element (2: bf16, 4: fp32).  Walks all lanes' chunks of 16 bytes
// in steps of a 128-byte line, eight steps further than K, as the kernels' look-ahead does; prints the number of wrong offsets.
int main(int, char **v) {
    const int n = atoi(v[1]), len = atoi(v[2]), K = n * len, el = atoi(v[4]), per = 16 / el, step = 128 / el;
    const long long stride = atoll(v[3]);
    long long wrong = 0;
    for (int chunk = 0; chunk < 8; ++chunk) {
        grace::KSegWalk walk{chunk * per};
        for (int k0 = 0; k0 < (K + step - 1) / step * step + 8 * step; k0 += step) {
            const int k = k0 + chunk * per;
            const uint32_t add = el == 2 ? walk.next(k, K, len, stride, step) : walk.next(k, K, len, stride, step, el);
            const uint32_t row = 31u * (uint32_t)len * (uint32_t)el, got = grace::offset_with(row, add);
            const long long want = row + ((long long)(k / len) * (stride - len)) * el;
            wrong += k < K ? got != want : got < grace::NO_DATA;
            wrong += grace::offset_with(grace::NO_DATA, add) < grace::NO_DATA;
        }
    }
    printf("%lld\n", wrong);
}
"""


@pytest.mark.parametrize("n_seg,seg_len,stride,el", [
    (2, 1408, 2048 * 1408, 2), (3, 40, 520 * 40, 2), (2, 8, 64, 2), (4, 352, 2048 * 352, 2),
    (3, 4096, 123456 * 4096, 2),         # 3 GB of weights: the last segment starts below 2 GiB, its end lies beyond
    (2, 32768, 32760 * 32768, 2),        # 4 GB
    (129, 8, 1048568 * 8, 2),            # many short segments: the look-ahead passes 64 further ones
    (2, 1388, 1024 * 1388, 4), (3, 40, 520 * 40, 4), (2, 4, 32, 4), (3, 200, 1024 * 200, 4),
    (3, 4096, 61728 * 4096, 4), (2, 16384, 32760 * 16384, 4), (129, 4, 1048568 * 4, 4),
])
def test_offsets_along_k_segments(tmp_path, n_seg, seg_len, stride, el):
    assert (n_seg - 1) * stride * el < 2 ** 31       # what the launcher lets through
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe), str(n_seg), str(seg_len), str(stride), str(el)], check=True, capture_output=True, text=True)
    assert int(out.stdout) == 0


DIVISIONS = r"""
#include <cstdio>
#include <initializer_list>
#include "kseg_walk.h"
// wrong quotients of numbers below 2^31: those next to the multiples of every length, first ones, last ones and some between
int main() {
    long long wrong = 0;
    for (int e = 1; e < 31; ++e)
        for (int len : {(1 << e) - 1, 1 << e, (1 << e) + 1, (1 << e) + (1 << e) / 3, 4 * e, 1388 + 4 * e})
            if (len >= 2) {
                const grace::KSegDiv div(len);
                const long long most = 0x7fffffffll / len;
                for (long long q = 0; q <= most; q += 1 + (q > 40 && q < most - 40) * (most / 50))
                    for (long long k = q * len - 1; k <= q * len + 1; ++k)
                        if (k >= 0 && k <= 0x7fffffffll) wrong += div((int)k) != (unsigned)(k / len);
                wrong += div(0x7fffffff) != (unsigned)(0x7fffffff / len);
            }
    printf("%lld\n", wrong);
}
"""


def test_segment_numbers_by_multiplication(tmp_path):
    src, exe = tmp_path / "div.cpp", tmp_path / "div"
    src.write_text(DIVISIONS)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    assert int(subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout) == 0
