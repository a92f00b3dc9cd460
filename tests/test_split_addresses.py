"""The split kernel's addresses of the weights (csrc/split_address.h), compiled for the host and walked over: a lane that has a chunk reads
that one, a lane that has none is beyond the tensor's end, and the offset that the lanes share lies inside the tensor.  Host only."""
import shutil
import subprocess

import pytest

from paper_1808_05567_amd import build

WALK = r"""
#include <cstdio>
#include <initializer_list>
#include "split_address.h"
using namespace convmi;
// reads: the lane has a chunk, at byte `at`
static bool bad(unsigned lane, unsigned shared, bool reads, unsigned long long at, unsigned long long size)
{
    const unsigned long long sum = (unsigned long long)lane + shared;
    if (lane == kNoChunk) return reads;
    if (shared >= size) return true;
    return reads ? sum != at || at + 16 > size : sum < size;
}
int main()
{
    int n = 0;
    for (int Cb : {1, 2, 3, 4, 5, 7, 8, 9, 25, 71})
        for (int RS : {1, 7, 9, 25})
            for (int Kp : {4, 8, 36, 64, 100, 132}) {
                const unsigned long long size = 16ull * Cb * RS * Kp;
                for (int cb = 0; cb < Cb; cb += 4)
                    for (int tap = 0; tap < RS; ++tap)
                        for (int k = 0; k < (Kp + 31) / 32 * 32; ++k)
                            for (int e = 0; e < 4; ++e) {
                                const int h = e >> 1, b = e & 1, blk = cb + e;
                                if (bad(weight_lane(k, h, b, Cb, RS, Kp), weight_shared(cb, tap, RS, Kp), blk < Cb && k < Kp, 16ull * (((unsigned long long)blk * RS + tap) * Kp + k), size)) {
                                    printf("Cb %d RS %d Kp %d: block %d tap %d row %d\n", Cb, RS, Kp, blk, tap, k);
                                    return 1;
                                }
                                ++n;
                            }
                for (int cb = 0; cb < Cb; cb += 4)
                    for (int tap = 0; tap < RS; ++tap)
                        for (int blk = 0; blk < (Kp / 4 + 7) / 8 * 8; ++blk)
                            for (int c = 0; c < 16 && 4 * cb + c < 4 * Cb; ++c) {
                                const bool reads = blk < Kp / 4;
                                if (bad(weight_lane_fwd(blk, c, Cb, RS, Kp), weight_shared_fwd(cb, tap, Cb), reads, 16ull * (((unsigned long long)blk * RS + tap) * 4 * Cb + 4 * cb + c), size)) {
                                    printf("forward weights, Cb %d taps %d Kp %d: rows %d tap %d channel %d\n", Cb, RS, Kp, blk, tap, 4 * cb + c);
                                    return 1;
                                }
                                ++n;
                            }
            }
    printf("%d\n", n);
    return 0;
}
"""


@pytest.mark.skipif(not shutil.which("g++"), reason="no host compiler")
def test_weights_are_read_inside_their_tensor(tmp_path):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(WALK)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I", build.CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    assert int(r.stdout) > 1000000
