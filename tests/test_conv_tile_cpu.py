"""Schedules of the convolution kernel that stages a window of input positions, on the CPU: the header that makes them,
compiled by the host compiler and walked over every tile, column and filter tap of small geometries.  Every column
belongs to one tile, every position a tap reads lies in the tile's window, and the window lies in the plane and in the
LDS rows that were set aside for it."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2311_14272_amd", "csrc")

HARNESS = r"""
#define __host__
#define __device__
#define __forceinline__ inline
#include <algorithm>
#include <vector>
#include <cstdio>
using std::min;
using std::max;
#include "conv_tile_plan.h"
using namespace crisp;
static long long bad, walked;
static void fail(const char* what, const ConvShape& a, const ConvTileSched& s, int tile) {
    if (++bad <= 5)
        printf("%s: H %d W %d kh %d kw %d stride %d pad %d Ncol %lld Sb %d, RG %d PT %d NC2 %d unit %d tile %d\n", what, a.H, a.W, a.kh, a.kw,
               a.stride, a.pad, (long long)a.Ncol, a.Sb, s.RG, s.PT, s.NC2, s.unit, tile);
}
static int by(int n, DivBy d) { return d.m ? (int)(((uint64_t)(uint32_t)n * d.m >> 32) >> d.shift) : n; }
static void walk(const ConvShape& a, const ConvTileSched& s) {
    const int HoWo = a.Ho * a.Wo;
    std::vector<char> seen((size_t)a.Ncol, 0);
    if (s.lds_bytes < 2 * s.HP * s.pitch + 128 + s.RG * (s.list_cap * 8 + s.chunks * 4) || s.lds_bytes > CONV_TILE_MAX_LDS) fail("LDS", a, s, -1);
    if (s.pitch < s.CC * 2 || s.pitch % 32 != 16) fail("pitch", a, s, -1);
    if (a.C % a.B) {                                          // block columns of several taps: one chunk and a table of octets
        if (s.octets * 8 != a.Kb * a.B || s.octets * 8 < a.kh * a.kw * a.C || (s.chunks > 1 && s.CC % 16)) fail("octets", a, s, -1);
        if (s.chunks * s.CC < a.C || (s.chunks - 1) * s.CC >= a.C) fail("chunks", a, s, -1);
        if ((int64_t)((a.kh - 1) * a.W + a.kw) / 2 * s.pitch + s.CC * 2 >= 1 << 20) fail("place", a, s, -1);
        if (s.lds_bytes < 2 * s.HP * s.pitch + 128 + s.RG * (s.list_cap * 8 + s.chunks * 4) + s.octets * 4) fail("LDS", a, s, -1);
        int entries = 2;                                     // what the kernel lists, every block kept
        for (int q = 0; q < s.chunks; ++q) {
            int run = 0;
            for (int bj = 0; bj < a.Kb; ++bj) {
                bool any = false;
                for (int k = bj * a.B; k < (bj + 1) * a.B && k < a.kh * a.kw * a.C; k += 8) any = any || k % a.C / s.CC == q;
                run += any;
            }
            entries += run + (run & 1);
        }
        if (entries > s.list_cap) fail("list", a, s, -1);
    } else if (s.octets || s.CC != s.CBC * a.B || s.chunks * s.CBC < s.CB || (s.chunks - 1) * s.CBC >= s.CB || s.CB * a.B != a.C) {
        fail("chunks", a, s, -1);
    }
    if (s.list_cap < a.Kb + s.chunks + 2 || s.row_groups * s.RG < a.Sb) fail("rows", a, s, -1);
    for (int tile = 0; tile < s.tiles; ++tile) {
        const int un = tile / s.per_unit;
        if (un != by(tile, div_by(s.per_unit))) fail("division", a, s, tile);
        const int first = un * s.unit + (tile - un * s.per_unit) * s.TC;
        const int end = min(min(first + s.TC, (un + 1) * s.unit), (int)a.Ncol);
        if (first >= end) continue;                          // an empty tile stages and stores nothing
        if ((first & 1) || ((end & 1) && end != a.Ncol) || end - first > 64 * s.NC2 * s.PT) { fail("columns", a, s, tile); continue; }
        const int row0 = by(first, div_by(a.Wo)), row1 = by(end - 1, div_by(a.Wo));
        if (row0 != first / a.Wo || row1 != (end - 1) / a.Wo) fail("division", a, s, tile);
        int lo = 0, npos = 0;
        conv_tile_window_of(a.H, a.W, a.kh, a.stride, a.pad, a.Ho, row0, row1, row0 / a.Ho, row1 / a.Ho, &lo, &npos);
        if (lo < 0 || npos < 4 || npos > 2 * s.HP || lo + npos > a.plane) { fail("window", a, s, tile); continue; }
        for (int col = first; col < end; ++col) {
            if (seen[col]++) fail("column twice", a, s, tile);
            const int img = col / HoWo, oh = (col - img * HoWo) / a.Wo, ow = col % a.Wo;
            for (int p = 0; p < a.kh; ++p) for (int q = 0; q < a.kw; ++q) {
                const int ih = oh * a.stride + p - a.pad, iw = ow * a.stride + q - a.pad;
                if (ih < 0 || ih >= a.H || iw < 0 || iw >= a.W) continue;
                const int pos = (img * a.H + ih) * a.W + iw - lo;
                if (pos < 0 || pos >= npos) fail("position", a, s, tile);
                // the kernel's form of the same place: the first tap's position for an even or an odd shift, plus half the shift
                const int base = (img * a.H + oh * a.stride - a.pad) * a.W + ow * a.stride - a.pad - lo, shift = p * a.W + q;
                const int even = (base & 1) * s.HP + (base >> 1), odd = ((base + 1) & 1) * s.HP + ((base + 1) >> 1);
                if (((shift & 1) ? odd : even) + (shift >> 1) != (pos & 1) * s.HP + (pos >> 1)) fail("row", a, s, tile);
                ++walked;
            }
        }
    }
    for (int col = 0; col < a.Ncol; ++col) if (!seen[col]) { fail("column missing", a, s, -1); break; }
}
int main() {
    for (int d = 1; d < 5000; ++d) for (int n : {0, 1, d - 1, d, d + 1, 1000003, 2147483646, 2147483647, 2147483647 / d * d, 2147483647 / d * d - 1})
        if (n >= 0 && by(n, div_by(d)) != n / d) { printf("%d / %d\n", n, d); ++bad; }
    for (int H = 1; H <= 15; H += 2) for (int W = 4; W <= 14; W += H == 7 || H == 13 ? 1 : 3) for (int batch : {1, 2, 13})
    for (int kh = 1; kh <= 5; kh += 2) for (int kw = 1; kw <= 5; kw += 2) for (int stride = 1; stride <= 3; ++stride) for (int pad = 0; pad < kh; ++pad) {
        if (H + 2 * pad < kh || W + 2 * pad < kw) continue;
        ConvShape a;
        a.n = 2; a.m = 8;
        a.H = H; a.W = W; a.kh = kh; a.kw = kw; a.stride = stride; a.pad = pad;
        a.Ho = (H + 2 * pad - kh) / stride + 1; a.Wo = (W + 2 * pad - kw) / stride + 1;
        a.Ncol = (int64_t)batch * a.Ho * a.Wo; a.plane = (int64_t)batch * H * W;
        for (int C : {8, 32, 40, 200, 1024}) for (int Sb : {1, 3, 9}) {
            a.B = C == 32 ? 32 : 64; a.C = C; a.Sb = Sb; a.Kb = (kh * kw * C + a.B - 1) / a.B;
            if (!conv_tile_covers(a)) continue;
            ConvTileSched s;
            double cost = 0;
            if (conv_tile_choose(a, (a.Kb + 1) / 2, &s, &cost)) walk(a, s);
            if (Sb == 3 && C != 1024) {
                for (int images = 0; images <= 3; ++images) for (int NC2 = 1; NC2 <= 2; ++NC2) for (int PT = 1; PT <= 8; PT *= 8)
                    if (conv_tile_plan(a, 1, PT, NC2, images, CONV_TILE_MAX_LDS, &s)) walk(a, s);
            }
        }
    }
    printf("%lld bad of %lld\n", bad, walked);
    return bad != 0 || walked == 0;
}
"""


def test_every_position_lies_in_the_window(tmp_path):
    src = tmp_path / "walk.cpp"
    src.write_text(HARNESS)
    exe = tmp_path / "walk"
    subprocess.run(["g++", "-O2", "-std=c++17", "-I" + CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout
