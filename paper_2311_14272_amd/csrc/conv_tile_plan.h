// Schedule of the convolution kernel that keeps a window of input positions in LDS (conv_tile.h): which output columns a
// workgroup takes, how many input positions it stages for them, and which of the possible schedules is taken.
// Integer and double arithmetic only, so that it also runs in a host test.
#pragma once
#include <cstdint>

namespace crisp {

constexpr int CONV_TILE_MAX_LDS = 152 * 1024;    // of 160 KB: the selector table of 4:8 is beside it
constexpr int CONV_TILE_MAX_KB = 512;            // block columns (taps x channel blocks)
constexpr int CONV_TILE_MAX_TAPS = 32;           // bits of a lane's tap mask; the last one is no tap: an octet that lies elsewhere
constexpr int CONV_TILE_MAX_WINDOW = 4096;       // positions staged at once

// The convolution as the schedule sees it.
struct ConvShape {
    int Sb, n, m, B, Kb;                         // block-rows, pattern, block edge, block columns
    int64_t Ncol, plane;                         // output columns, elements of one channel plane
    int C, H, W, kh, kw, stride, pad, Ho, Wo;
};

// n / d for 0 <= n < 2^31 by a multiplication: m = ceil(2^(31 + l) / d), 2^(l - 1) < d <= 2^l (m = 0: d is 1).
struct DivBy {
    uint32_t m;
    int shift;
};
inline DivBy div_by(int d) {
    int l = 0;
    while (((int64_t)1 << l) < d) ++l;
    if (l == 0) return DivBy{0u, 0};
    return DivBy{(uint32_t)((((uint64_t)1 << (31 + l)) + (uint64_t)d - 1) / (uint64_t)d), l - 1};
}

struct ConvTileSched {
    int RG, PT;              // block-rows and column parts per workgroup: RG * PT waves
    int NC2;                 // column pairs of tiles per wave: 64 * NC2 columns
    int row_groups;          // groups of RG block-rows
    int unit, per_unit, TC;  // tile t starts at column (t / per_unit) * unit + (t % per_unit) * TC and ends with its unit
    int tiles;
    int CC, CB, CBC, chunks; // channels per chunk; channel blocks in all and per chunk
    int kh;
    int HP;                  // LDS rows of even positions (as many for the odd ones)
    int pitch;               // bytes of an LDS row
    int list_cap;            // entries of a block-row's list
    int octets;              // octets of K-rows (rounded up to whole blocks) where a block column holds several taps, else 0
    int lds_bytes;
    DivBy by_Wo, by_Ho, by_unit;   // output width and height, tiles per unit
};

// The input positions [lo, lo + npos) of the plane that the output columns [col_first, col_end) touch: whole input rows,
// from a multiple of four on.
__host__ __device__ __forceinline__ void conv_tile_window_of(int H, int W, int kh, int stride, int pad, int Ho, int row0, int row1, int img0, int img1,
                                                            int* lo, int* npos) {
    const int oh0 = row0 - img0 * Ho, oh1 = row1 - img1 * Ho;
    const int ih0 = min(max(oh0 * stride - pad, 0), H - 1);
    const int ih1 = min(max(oh1 * stride - pad + kh - 1, 0), H - 1);
    *lo = ((img0 * H + ih0) * W) & ~3;
    *npos = (img1 * H + ih1 + 1) * W - *lo;
}

// Input positions a tile touches at most, from its output rows (of images laid end to end).  The padding is smaller than
// the filter, so the first input row of a window lies before the image's end and its last one behind the image's start.
inline int64_t conv_tile_window(const ConvShape& a, int64_t rows, bool crosses) {
    int64_t span = (rows - 1) * a.stride + a.kh;
    if (crosses && a.H > a.stride * a.Ho) span += (rows + a.Ho - 2) / a.Ho * (a.H - a.stride * a.Ho);
    if (!crosses && span > a.H) span = a.H;
    return span * a.W + 3;                        // + 3: the window begins at a multiple of four
}

// Schedule with RG x PT waves of 64 * NC2 columns; images > 0: tiles are whole images (images of them) or equal parts
// of one (images 1, a part is then at most the workgroup's columns); images 0: runs of columns across images.
// False if it does not apply or fit.  (32-bit arithmetic: it is done for several schedules on every call.)
inline bool conv_tile_plan(const ConvShape& a, int RG, int PT, int NC2, int images, int max_lds, ConvTileSched* out) {
    ConvTileSched& s = *out;
    const unsigned cols = 64u * NC2 * PT, Ncol = (unsigned)a.Ncol, Wo = (unsigned)a.Wo;
    s.RG = RG; s.PT = PT; s.NC2 = NC2; s.kh = a.kh;
    s.row_groups = (int)(((unsigned)a.Sb + RG - 1) / (unsigned)RG);
    int64_t window;
    if (images == 0) {
        s.TC = (int)cols; s.per_unit = 1 << 30; s.unit = 1 << 30;
        window = conv_tile_window(a, (cols + Wo - 2) / Wo + 1, true);
        s.tiles = (int)((Ncol + cols - 1) / cols);
    } else {
        const unsigned unit = Wo * (unsigned)a.Ho * (unsigned)images;
        if (unit & 1) return false;               // a lane's two columns stay in one tile
        if (images > 1 && unit > cols) return false;
        s.per_unit = (int)((unit + cols - 1) / cols);
        s.TC = (int)((unit + s.per_unit - 1) / (unsigned)s.per_unit);
        s.TC += s.TC & 1;
        s.unit = (int)unit;
        window = s.per_unit == 1 ? (int64_t)images * a.H * a.W + 3 : conv_tile_window(a, ((unsigned)s.TC + Wo - 2) / Wo + 1, false);
        s.tiles = (int)((Ncol + unit - 1) / unit) * s.per_unit;
    }
    if (window > CONV_TILE_MAX_WINDOW) return false;
    s.HP = (int)(window + 1) / 2;
    if ((unsigned)a.C % (unsigned)a.B != 0) {
        // block columns that span taps: chunks of whole staging units, and a table of the octets of K-rows
        s.CB = s.CBC = a.Kb;
        s.octets = a.Kb * (a.B / 8);
        const int most = ((max_lds - 144 - s.octets * 4 - RG * 8 * (a.Kb + 4)) / (2 * s.HP) - 16) / 32 * 16 - 16;
        if (most < 16) return false;
        s.chunks = a.C <= most ? 1 : (a.C + most - 1) / most;
        s.CC = s.chunks == 1 ? a.C : (a.C + s.chunks * 16 - 1) / (s.chunks * 16) * 16;
        s.chunks = (a.C + s.CC - 1) / s.CC;
        s.pitch = ((s.CC + 7) / 8 | 1) * 16;
        if ((int64_t)(a.kh * a.W / 2 + 1) * s.pitch >= (1 << 20)) return false;      // a place has 20 bits in the table
    } else {
        s.CB = (int)((unsigned)a.C / (unsigned)a.B);
        s.octets = 0;
        const int fixed = 128 + RG * 8 * (a.Kb + 2 * s.CB + 4);
        // as many channel blocks per chunk as fit, evenly
        int cbc = ((max_lds - fixed) / (2 * s.HP) - 16) / (a.B * 2);
        if (cbc < 1) return false;
        if (cbc >= s.CB) {
            s.CBC = s.CB;
            s.chunks = 1;
        } else {
            s.chunks = (s.CB + cbc - 1) / cbc;
            s.CBC = (s.CB + s.chunks - 1) / s.chunks;
            s.chunks = (s.CB + s.CBC - 1) / s.CBC;
        }
        s.CC = s.CBC * a.B;
        s.pitch = s.CC * 2 + 16;
    }
    // (a block that spans taps is walked in every chunk it has a part in: at most one more entry per tap and chunk)
    s.list_cap = a.Kb + s.chunks + 2 + (s.octets && s.chunks > 1 ? a.kh * a.kw * s.chunks : 0);
    s.lds_bytes = (2 * s.HP * s.pitch + 128 + RG * (s.list_cap * 8 + s.chunks * 4) + s.octets * 4 + 15) / 16 * 16;
    return s.lds_bytes <= max_lds;
}

// What the kernel takes at all.
inline bool conv_tile_covers(const ConvShape& a) {
    return a.B >= 32 && a.C % 8 == 0 && a.kh * a.kw < CONV_TILE_MAX_TAPS && a.Kb <= CONV_TILE_MAX_KB && a.W >= 4 &&
           a.pad < a.kh && a.plane < ((int64_t)1 << 26) && a.Ncol < ((int64_t)1 << 30);
}

// Waves of a compute unit that the kernel's registers leave room for.  2:4 with 64x64 blocks has two packed slices of 20
// registers on their way: three waves per SIMD would spill 14 to 54 of 168 registers (256 x 10400 x 20384: 190 us, with two
// waves 104; fifteen such convolutions with channels that are no multiple of 64 at 0.57 of the time, twenty others at 0.98).
// 3:4, 4:4 and 8:8 spill 6 to 17 of 168: with two waves and nothing spilled 1.000 of the time over 900, so three stay.
constexpr int conv_tile_waves(int n, int m, int B, int NC2) { return NC2 == 2 || (n == 2 && m == 4 && B == 64) ? 8 : 12; }

// What a schedule has a compute unit do, in clocks.
struct ConvTileClocks {
    int waves, per_cu;       // waves of a workgroup, workgroups of a compute unit
    double matrix, vector;   // of one kept block in one wave
};
inline ConvTileClocks conv_tile_clocks(const ConvShape& a, const ConvTileSched& s) {
    ConvTileClocks c;
    c.waves = s.RG * s.PT;
    const int fit = 160 * 1024 / (s.lds_bytes + 4352), room = conv_tile_waves(a.n, a.m, a.B, s.NC2) / c.waves;
    c.per_cu = fit < room ? fit : room;
    c.matrix = (a.n <= 2 ? 256.0 : 512.0) * s.NC2 * (a.B == 64 ? 1.0 : 0.25);
    c.vector = (a.n == 3 ? 1300.0 : a.n == 4 && a.m == 8 ? 450.0 : a.n == 2 && a.m == 8 ? 430.0 : 200.0) * (a.B == 64 ? 1.0 : 0.3) + 60.0 * s.NC2 +
               (s.octets ? (a.B == 64 ? 128.0 : 64.0) * s.NC2 : 0.0);
    return c;
}

// Estimated time of a schedule in clocks of a compute unit, by which one of them is chosen (bpr: kept blocks per block-row;
// bf16 outputs, so that the choice and with it the order of the sums is the same for both output types).  A workgroup's
// phases follow one another: window in (9 bytes per clock and compute unit when all stage at once: 5 TB/s), blocks, rows
// out; two and more workgroups of a compute unit overlap theirs.
inline double conv_tile_cost(const ConvShape& a, const ConvTileSched& s, int bpr) {
    const ConvTileClocks c = conv_tile_clocks(a, s);
    const int per_cu = c.per_cu, wgs = s.tiles * s.row_groups;
    const double block = c.waves / 4.0 * (c.matrix + 0.5 * c.vector);
    const double in = 2.0 * s.HP * a.C * 2 / 9.0 + 3000.0 * s.chunks;
    const double out = (double)(s.RG < a.Sb ? s.RG : a.Sb) * a.B * s.TC * 2 / 9.0;
    const double walk = bpr * block * (1.0 + 0.12 * (s.chunks - 1)) * (s.octets && s.chunks > 1 ? 1.0 + (double)a.B / s.CC : 1.0);
    const double mem = in + out, rounds = (double)(((unsigned)wgs + 256u * per_cu - 1) / (256u * per_cu));
    const double one = per_cu == 1 ? mem + walk : (mem > walk ? mem * per_cu + walk : walk * per_cu + mem);
    return rounds * (5000.0 + one);
}

// The schedule of least estimated time; false where none applies.
inline bool conv_tile_choose(const ConvShape& a, int bpr, ConvTileSched* out, double* cost) {
    double best = 0.0;
    const unsigned HoWo = (unsigned)a.Ho * (unsigned)a.Wo;
    const int rg = a.Sb > 4 ? 8 : a.Sb > 2 ? 4 : a.Sb;
    for (int RG = rg; RG >= 1 && RG * 2 >= rg && (RG == rg || RG == 4); RG /= 2) {
        for (int NW = RG == 8 ? 8 : 4; NW <= 8; NW *= 2) {
            for (int NC2 = 1; NC2 <= 2; ++NC2) {
                const unsigned cols = 64u * NC2 * (NW / RG);
                for (int way = 0; way < 2; ++way) {
                    int images = 0;
                    if (way == 1) {
                        images = HoWo * 2 > cols ? 1 : (int)(cols / HoWo);
                        if (HoWo & images & 1) images -= images > 1;
                    }
                    ConvTileSched s;
                    if (!conv_tile_plan(a, RG, NW / RG, NC2, images, CONV_TILE_MAX_LDS, &s)) continue;
                    const double c = conv_tile_cost(a, s, bpr);
                    if (best == 0.0 || c < best) { best = c; *out = s; }
                }
            }
        }
    }
    *cost = best;
    if (best == 0.0) return false;
    out->by_Wo = div_by(a.Wo); out->by_Ho = div_by(a.Ho); out->by_unit = div_by(out->per_unit);
    return true;
}

}  // namespace crisp
