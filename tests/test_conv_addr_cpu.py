"""Addresses of the fused lowering on the CPU: the header that computes them, compiled by the host compiler and walked
over every output pair and filter tap of small geometries.  Every load has to lie inside the channel plane and every
element that is selected has to be the lowering's."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2311_14272_amd", "csrc")

HARNESS = r"""
#define __host__
#define __device__
#define __forceinline__ inline
#include <algorithm>
using std::min;
#include "conv_addr.h"
#include <cstdio>
using namespace crisp;
static long long outside, wrong, pairs;
static void report(const char* what, int mode, int H, int W, int batch, int kh, int kw, int stride, int pad, int col, int a, int b) {
    if (outside + wrong <= 5)
        printf("%s: mode %d H %d W %d batch %d k %dx%d stride %d pad %d column %d tap (%d, %d)\n", what, mode, H, W, batch, kh, kw, stride, pad, col, a, b);
}
int main() {
    for (int H = 1; H <= 6; ++H) for (int W = 1; W <= 9; ++W) for (int batch = 1; batch <= 2; ++batch)
    for (int kh = 1; kh <= 7; ++kh) for (int kw = 1; kw <= 7; ++kw) for (int stride = 1; stride <= 3; ++stride) for (int pad = 0; pad <= 5; ++pad) {
        if (H + 2 * pad < kh || W + 2 * pad < kw) continue;
        const int Ho = (H + 2 * pad - kh) / stride + 1, Wo = (W + 2 * pad - kw) / stride + 1;
        const int ncol = batch * Ho * Wo, plane = batch * H * W;
        if (ncol & 1) continue;
        const bool same_pad = kh == 2 * pad + 1 && kw == 2 * pad + 1;
        const bool one = stride == 1 && ((Wo & 1) == 0 || same_pad) && W >= 2 && Wo >= 2;      // the host's rule for mode 1
        for (int mode = one ? 1 : 2; mode <= 2; ++mode)
        for (int col = 0; col < ncol; col += 2) for (int a = 0; a < kh; ++a) for (int b = 0; b < kw; ++b) {
            OutPos p[2];
            int want[2];
            for (int c = 0; c < 2; ++c) {
                const int t = (col + c) / Wo;
                p[c] = OutPos{t / Ho, t % Ho, (col + c) % Wo};
                const int ih = p[c].oh * stride + a - pad, iw = p[c].ow * stride + b - pad;
                want[c] = ih >= 0 && ih < H && iw >= 0 && iw < W ? (p[c].img * H + ih) * W + iw : -1;
            }
            ++pairs;
            int got[2];
            bool in;
            if (mode == 1) {
                const PairSource s = pair_one_load(H, W, pad, plane, p[0], p[1], a, b);
                in = s.off >= 0 && s.off + 2 <= plane;
                const uint32_t sel[2] = {s.sel_lo, s.sel_hi};
                for (int c = 0; c < 2; ++c) got[c] = sel[c] == SEL_ZERO ? -1 : s.off + (sel[c] == SEL_HI);
            } else {
                const PairSource s = pair_two_loads(H, W, pad, stride, plane, p[0], p[1], a, b);
                in = s.off >= 0 && s.off < plane && s.off2 >= 0 && s.off2 < plane;
                got[0] = s.sel_lo == SEL_ZERO ? -1 : s.off;
                got[1] = s.sel_hi == SEL_ZERO ? -1 : s.off2;
            }
            if (!in) { ++outside; report("outside the plane", mode, H, W, batch, kh, kw, stride, pad, col, a, b); }
            if (got[0] != want[0] || got[1] != want[1]) { ++wrong; report("wrong element", mode, H, W, batch, kh, kw, stride, pad, col, a, b); }
        }
    }
    printf("pairs %lld outside %lld wrong %lld\n", pairs, outside, wrong);
    return outside || wrong;
}
"""


def test_every_load_is_inside_its_plane_and_right(tmp_path):
    src = tmp_path / "walk.cpp"
    src.write_text(HARNESS)
    exe = str(tmp_path / "walk")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I" + CSRC, str(src), "-o", exe], check=True, timeout=120)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout
