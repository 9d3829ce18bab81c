"""Byte offsets of packed 16 x 16 blocks up to the largest layer that a descriptor may state (values just under 4 GiB): the
header that forms them, compiled by the host compiler with its checks for signed overflow, against 64-bit arithmetic."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2311_14272_amd", "csrc")

HARNESS = r"""
#define __host__
#define __device__
#define __forceinline__ inline
#include <cstdio>
#include <initializer_list>
#include "packed_addr.h"
using namespace crisp;
int main() {
    long long bad = 0, asked = 0;
    for (int m = 4; m <= 8; m += 4) for (int n = 1; n <= m; ++n) {
        const int slots = 16 / m * n, words = (slots * (m == 4 ? 2 : 3) + 31) / 32;
        const int64_t most = ((int64_t)1 << 32) / (16 * slots * 2) - 1;        // blocks below 4 GiB of values
        for (int64_t t : {(int64_t)0, most / 3, most / 2 - 1, most / 2, most / 2 + 1, most * 2 / 3, most - 1})
            for (int row = 0; row < 16; ++row) for (int slot = 0; slot < slots; ++slot, ++asked) {
                bad += b16_value_at((int)t, row, slots, slot) != ((t * 16 + row) * slots + slot) * 2;
                bad += b16_words_at((int)t, row, words) != (t * 16 + row) * words * 4;
            }
    }
    printf("%lld bad of %lld\n", bad, asked);
    return bad != 0;
}
"""


def test_offsets_up_to_four_gigabytes(tmp_path):
    src = tmp_path / "at.cpp"
    src.write_text(HARNESS)
    exe = tmp_path / "at"
    subprocess.run(["g++", "-O1", "-std=c++17", "-fsanitize=signed-integer-overflow", "-fno-sanitize-recover=all", "-I" + CSRC, str(src), "-o",
                    str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
