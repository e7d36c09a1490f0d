"""The addresses of the unsigned char walk, enumerated on the host: every 16-byte read of every strip, row and lane,
taken from the header that the kernel computes them with, lies in the image's memory (H - 1 rows of the pitch and the W
bytes of the last), for widths around a strip's 256 columns, few and many rows and padded rows; rows as wide as a
strip's reads are clamped in the first and the last two only, and rows outside the image are clamped ones."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1605_06399_amd", "csrc")

PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include "u8_rows.hpp"
using namespace icl;

int main() {
    const int heights[] = {1, 2, 3, 4, 5, 6, 8, 12, 17, 18, 19, 20, 27, 40};
    const int pads[] = {0, 1, 3, 8, 100, 300};
    long long reads = 0;
    for (int W = 16; W <= 800; ++W)
        for (int H : heights)
            for (int pad : pads) {
                const unsigned sp = W + pad;
                const long long size = (long long)(H - 1) * sp + W;
                const int tail = u8_tail(W, H, sp);
                for (int xs = 0; xs < W; xs += U8_COLS) {
                    for (int q = -7; q < H + 30; ++q)
                        for (int lane = 0; lane < 64; ++lane) {
                            const int n = lane & 15, g = lane >> 4, c = u8_col(xs, n, g);
                            const int cb = std::min(std::max(c, 0), W - 16);
                            const long long at = (long long)u8_row(q, H) * sp + u8_lane(q, H, tail, g >> 1 ? sp : 0u, c, cb);
                            ++reads;
                            const bool wide_guarded = W >= U8_RIGHT && q >= 1 && q + 1 < H - 1 && u8_guarded(q, tail);
                            const bool outside_free = (q < 0 || q + 1 >= H) && !u8_guarded(q, tail);
                            if (at < 0 || at + 16 > size || (u8_inside(xs, W) && c != cb) || wide_guarded || outside_free) {
                                std::printf("W=%d H=%d pitch=%u strip %d row %d lane %d: bytes %lld..%lld of %lld\n", W, H, sp,
                                            xs, q, lane, at, at + 15, size);
                                return 1;
                            }
                        }
                }
            }
    std::printf("%lld reads\n", reads);
    return 0;
}
"""


@pytest.mark.skipif(not shutil.which("g++"), reason="needs a host C++ compiler")
def test_every_read_lies_in_the_image(tmp_path):
    src, exe = tmp_path / "rows.cpp", tmp_path / "rows"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    p = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert p.returncode == 0, p.stdout
