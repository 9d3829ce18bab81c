"""Estimated times of the ways to run a convolution, on the CPU: the header that forms them, compiled by the host compiler,
for convolutions that were timed every way.  Each estimate is within a factor of 1.8 of its time (four standard deviations of
the fit, 0.143 in the logarithm), and a way that was slower than the older one by a quarter and more is not ahead of it by the margin."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2311_14272_amd", "csrc")

# S, C, H, batch, k, stride, n, m, B, density; conv mode; lists split over four waves in the product over X / in the register
# kernels; us through X (0: not planned that way), from a window (0: not covered), in the register kernels (0: not covered)
CASES = [
    (256, 464, 28, 3, 5, 1, 1, 4, 32, 0.70, 3, 1, 1, 61.7, 100.1, 149.0),
    (75, 304, 20, 3, 1, 2, 4, 8, 64, 0.47, 3, 0, 0, 8.8, 0, 12.8),
    (960, 32, 20, 1, 3, 1, 4, 8, 64, 0.31, 3, 0, 0, 9.5, 9.4, 13.3),
    (448, 200, 28, 200, 1, 2, 4, 8, 64, 0.41, 3, 0, 0, 43.3, 0, 51.5),
    (839, 64, 7, 91, 3, 2, 4, 8, 64, 0.74, 2, 1, 1, 14.3, 17.9, 12.7),
    (508, 64, 20, 18, 3, 2, 2, 4, 64, 0.77, 2, 1, 1, 0, 15.0, 8.1),
    (256, 192, 20, 18, 5, 1, 2, 8, 64, 0.32, 1, 1, 1, 0, 26.5, 16.5),
    (64, 304, 13, 66, 5, 1, 2, 8, 64, 0.20, 3, 1, 1, 0, 36.1, 26.0),
    (200, 448, 7, 80, 3, 1, 1, 4, 64, 0.79, 1, 1, 1, 0, 25.5, 20.1),
    (512, 512, 14, 256, 3, 2, 4, 8, 64, 0.40, 2, 0, 0, 130.0, 55.0, 0),
]

HARNESS = r"""
#define __host__
#define __device__
#define __forceinline__ inline
#include <algorithm>
#include <cstdio>
#include <cstdlib>
using std::min;
using std::max;
#include "conv_ways.h"
using namespace crisp;
static int bad;
static void near(const char* what, double us, double est) {
    printf(" %s %.1f (%.1f)", what, us, est);
    if (us > 0.0 && (est > us * 1.8 || us > est * 1.8)) { printf(" FAR"); ++bad; }
}
int main() {
    int S, C, H, batch, k, stride, n, m, B, mode, sx, sr;
    double d, x, window, reg;
    while (scanf("%d %d %d %d %d %d %d %d %d %lf %d %d %d %lf %lf %lf", &S, &C, &H, &batch, &k, &stride, &n, &m, &B, &d, &mode, &sx, &sr, &x, &window, &reg) == 16) {
        ConvShape a;
        a.Sb = (S + B - 1) / B; a.n = n; a.m = m; a.B = B; a.C = C; a.H = a.W = H; a.kh = a.kw = k; a.stride = stride; a.pad = k / 2;
        a.Kb = (k * k * C + B - 1) / B; a.Ho = a.Wo = (H + 2 * a.pad - k) / stride + 1;
        a.Ncol = (int64_t)batch * a.Ho * a.Wo; a.plane = (int64_t)batch * H * H;
        const int bpr = max(1, (int)(d * a.Kb + 0.5));
        ConvTileSched s;
        double clocks = 0.0;
        const bool covers = k > 1 && conv_tile_covers(a) && conv_tile_choose(a, bpr, &s, &clocks);
        const double ex = conv_x_us(a, bpr, sx, n <= 2), ew = covers ? conv_tile_us(a, s, bpr) : 0.0, er = conv_reg_us(a, bpr, sr, mode);
        printf("%d x %d x %d:", S, k * k * C, (int)a.Ncol);
        near("x", x, ex); near("window", window, ew); near("reg", reg, er);
        if (covers && (ew < WINDOW_LEAST_US || !(ew < 1e9))) ++bad;
        if (x > 0.0 && window > x * 1.25 && ew * WINDOW_OVER_X < ex) { printf(" window over X"); ++bad; }
        if (x > 0.0 && reg > x * 1.15 && er * REG_OVER_X < ex && bpr <= 8) { printf(" register kernels over X"); ++bad; }
        if (x == 0.0 && window > reg * 1.25 && ew * WINDOW_OVER_FUSED < er) { printf(" window over register kernels"); ++bad; }
        if (x > 0.0 && window > 0.0 && window < x * 0.6 && !(ew * WINDOW_OVER_X < ex)) { printf(" X over window"); ++bad; }
        printf("\n");
    }
    return bad != 0;
}
"""


def test_estimates_of_timed_convolutions(tmp_path):
    src = tmp_path / "ways.cpp"
    src.write_text(HARNESS)
    exe = tmp_path / "ways"
    subprocess.run(["g++", "-O2", "-std=c++17", "-I" + CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], input="\n".join(" ".join(str(v) for v in c) for c in CASES), capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
    assert len(r.stdout.splitlines()) == len(CASES)
