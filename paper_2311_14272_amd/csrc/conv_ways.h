// Estimated times of the ways a convolution may be run, in microseconds: which of them is taken is decided on these.
//
// Sums of a few terms whose weights were fitted (least squares of the relative error) to 6500 random convolutions, each
// timed every way that takes it: 3x3 and 5x5 filters at stride 1 and 2, strided 1x1, 16 to 512 channels of any count, 24 to
// 1024 outputs, images of 7x7 to 56x56, batch 1 to 256 (up to 3 GB of X), all patterns, both block sizes, densities 0.2 to
// 0.8, both output types, odd numbers of columns.  An estimate is off by a factor of 1.15 (one standard deviation), so a
// way that is not the older one of two has to be the faster one by the margins below.  Outputs count as bf16: the choice,
// and with it the order of the sums, is then the same for both output types.
// Double arithmetic only, so that it also runs in a host test.
#pragma once
#include "conv_tile_plan.h"

namespace crisp {

// By how much an estimate has to be ahead.  4776 convolutions that the weights were not fitted to: the 2296 planned through
// X with rows of equal length run at 0.764 of the time that X takes (geometric mean; 0.740 with the best of all ways each
// time), five are slower by more than 5 % (1.15 the worst: 986 x 1584 x 20384 2:8 78 / 90 us); the 1480 planned fused at
// 0.878 of the older fused kernels' (0.847 at best), three are slower (669 x 4032 x 9408 3:4 103 / 137 us).  With margins of
// 1.1 the means are 0.01 lower and ten times as many are slower, up to 1.5.  Where K is short (8 or 16 channels, K <= 192) the
// estimates are at their worst: 69 that run in the window kernel at 0.72, seven slower by more than 5 % (480 x 144 x 68992 4:4
// 35 / 46 us); a further margin of 1.25 there loses more (0.806 -> 0.827 over 900) than it mends (ten slower by a tenth, then eight).
constexpr double WINDOW_OVER_X = 1.25, REG_OVER_X = 1.25, WINDOW_OVER_FUSED = 1.25;
// ... and once more where block-rows differ in length: a workgroup of the window kernel lasts as long as its longest row, X
// is multiplied by a kernel that deals the blocks evenly.  1000 planned through X and pruned over the whole grid, half of
// them with block-rows of unequal importance: 0.888, four slower by more than 5 % (256 x 5200 x 9408 4:8 77 / 104 us); without
// it 0.87, 17, and up to 1.6.
constexpr double WINDOW_UNEVEN = 1.4;

inline bool dense_expansion(const ConvShape& a) { return a.n > 2; }
// Kept blocks x 64 columns per compute unit; a 32 x 32 block counts a third.
inline double block_tiles(const ConvShape& a, int bpr) {
    return (double)a.Sb * (double)((a.Ncol + 63) / 64) * bpr / 256.0 * (a.B == 64 ? 1.0 : 0.3);
}
inline double output_mb(const ConvShape& a) { return (double)a.Sb * a.B * (double)a.Ncol * 2e-6; }
// Blocks that one wave walks one after the other (split: four waves share a block-row's list), in 64 x 64 blocks.
inline double block_chain(const ConvShape& a, int bpr, bool split) { return (split ? (bpr + 3) / 4 : bpr) * (a.B == 64 ? 1.0 : 0.5); }

// X written and read (MB), the product's blocks and its longest chain.  sparse: the product's matrix-core instruction.
inline double conv_x_us(const ConvShape& a, int bpr, bool split, bool sparse) {
    const double x = (double)a.kh * a.kw * a.C * (double)a.Ncol * 4e-6;
    return 8.0 + (a.kh * a.kw > 1 ? 0.2 : 0.28) * x + 0.2 * output_mb(a) +
           block_tiles(a, bpr) * (0.17 + (sparse ? 0.0 : 0.085) + (a.B == 64 ? 0.0 : 0.12)) + 1.65 * block_chain(a, bpr, split);
}

// The register kernels, by how they find their columns (conv modes 1 to 4: pairs from one load, one by one, every K-row on
// its own, 8-byte pieces of a strided row).  Past 20 blocks x 64 columns per compute unit the caches no longer help.
inline double conv_reg_us(const ConvShape& a, int bpr, bool split, int mode) {
    const double bt = block_tiles(a, bpr), many = bt > 20.0 ? bt - 20.0 : 0.0, chain = block_chain(a, bpr, split), y = output_mb(a);
    const double d = dense_expansion(a) ? 1.0 : 0.0;
    const bool b64 = a.B == 64;
    switch (mode) {
        case 1: return 4.0 + bt * ((b64 ? 0.13 : 0.23) + 0.05 * d) + chain * (0.9 + 0.18 * d) + 0.18 * y + 0.1 * many;
        case 2: return 4.0 + bt * ((b64 ? 0.3 : 0.78) + 0.06 * d) + chain * (1.7 + 0.15 * d) + 0.26 * y + 0.25 * many;
        case 3: return 3.2 + bt * (b64 ? 0.32 + 0.31 * d : 0.59 + 0.08 * d) + chain * (b64 ? 3.7 + 1.3 * d : 2.6) + 0.2 * y + 0.25 * many;
        default: return 4.6 + bt * ((b64 ? 0.37 : 0.74) + 0.15 * d) + chain * (0.6 + 0.3 * d) + 0.15 * y + 0.25 * many;
    }
}

// The kernel that stages whole output rows (conv_lds.h) where its rule takes it, and the one for few channels.
inline double conv_staged_us(const ConvShape& a, int bpr) {
    const double bt = block_tiles(a, bpr), d = dense_expansion(a) ? 1.0 : 0.0;
    if (a.stride == 1) return 4.5 + bt * (0.09 + 0.11 * d) + 0.28 * output_mb(a) + 0.12 * a.C * (double)a.plane * 2e-6 + 0.4 * bpr + a.C / 32.0;
    return 8.0 + bt * (0.23 + 0.05 * d) + 0.2 * output_mb(a) + 0.5 * bpr;
}
inline double conv_patch_us(const ConvShape& a, int bpr) { return 22.0 + 0.4 * block_tiles(a, bpr); }

// The least that the next estimate comes to: what is not ahead of anything else by that needs no schedule looked for (0.1 of
// the 3.4 us of host time of a small convolution's call).
constexpr double WINDOW_LEAST_US = 6.0;

// The window kernel with schedule s: rounds of workgroups, in each of them window in, blocks (matrix and vector
// instructions in clocks, and a wave's wait per block) and rows out.
inline double conv_tile_us(const ConvShape& a, const ConvTileSched& s, int bpr) {
    const ConvTileClocks c = conv_tile_clocks(a, s);
    const double wgs = (double)s.tiles * s.row_groups;
    int per_cu = c.per_cu, rounds = 1;
    if (wgs > 256.0 * per_cu) rounds = (int)((wgs + 256.0 * per_cu - 1.0) / (256.0 * per_cu));
    else if (wgs <= 256.0 * (per_cu - 1)) per_cu = wgs <= 256.0 ? 1 : (int)((wgs + 255.0) / 256.0);
    const bool spans = s.octets != 0;
    const double block = c.waves / 4.0 * (7e-4 * c.matrix + 1.4e-4 * c.vector);
    const double in = 1.15e-5 * 4.0 * s.HP * a.C, out = 2.8e-5 * (s.RG < a.Sb ? s.RG : a.Sb) * a.B * s.TC * 2.0;
    const double wait = spans ? 0.24 + (s.chunks > 1 ? 0.3 : 0.0) : 0.17;
    return WINDOW_LEAST_US + 6.0 * (rounds - 1) + rounds * (per_cu * (in + out + bpr * block) + bpr * wait + (spans ? 4.0 : 2.6) * (s.chunks - 1));
}

}  // namespace crisp
