// Where a lane's two output columns of one filter tap lie in the convolution's input (fused lowering, conv modes 1 and
// 2).  Offsets are elements inside a plane [batch][H][W] of one channel; the caller adds the channel and turns them into
// byte offsets of loads that nothing clips, so they have to stay inside the plane whatever the padding: a column outside
// the image is loaded from a place inside the plane and its selector yields zeros.
// Integer arithmetic only, so that it also runs on the host.
#pragma once
#include <cstdint>

namespace crisp {

constexpr uint32_t SEL_LO = 0x05040100u;    // r0.lo | r1.lo << 16
constexpr uint32_t SEL_HI = 0x07060302u;    // r0.hi | r1.hi << 16
constexpr uint32_t SEL_ZERO = 0x0C0C0C0Cu;  // v_perm_b32: selector byte 0x0c yields 0x00

// An output position (image, oh, ow).
struct OutPos {
    int img, oh, ow;
};
struct PairSource {
    int off, off2;              // off2: mode 2 only
    uint32_t sel_lo, sel_hi;
};

// Mode 1: the sources of the two columns are neighbours in memory when both are inside the image, and come from one load
// of the elements off, off + 1.  (The second column is the next output position, which may lie in the next output row or
// image, odd Wo.  The host picks this mode only where the two sources are then still neighbours: always inside one output
// row, and across rows and images when the padding is (k - 1) / 2 in both directions, because consecutive output
// positions then read consecutive input elements for every tap.)  plane >= 2 elements.
__host__ __device__ __forceinline__ PairSource pair_one_load(int H, int W, int pad, int plane, OutPos p0, OutPos p1, int a, int b) {
    const int ih = p0.oh + a - pad, iw = p0.ow + b - pad;
    const int ih1 = p1.oh + a - pad, iw1 = p1.ow + b - pad;
    const bool v0 = (unsigned)ih < (unsigned)H && (unsigned)iw < (unsigned)W;
    const bool v1 = (unsigned)ih1 < (unsigned)H && (unsigned)iw1 < (unsigned)W;
    // (the position itself as long as the padding is at most (k - 1) / 2; with more, output rows and columns go on past
    // the image's and the last of them would lie past the plane)
    const int centre = min((p0.img * H + p0.oh) * W + p0.ow, plane - 2);
    const int src = (p0.img * H + ih) * W + iw;
    const int src1 = (p1.img * H + ih1) * W + iw1;
    PairSource s = {centre, 0, SEL_ZERO, SEL_ZERO};
    if (v0 && v1) {
        s.off = src;
        s.sel_lo = SEL_LO;
        s.sel_hi = SEL_HI;
    } else if (v1) {
        // column 1 <- e0; at the very end of the plane the load starts one element earlier and column 1 <- e1
        const bool last = src1 + 1 >= plane;
        s.off = last ? src1 - 1 : src1;
        s.sel_hi = last ? SEL_HI : SEL_LO;
    } else if (v0) {
        // column 0 <- e1; for the plane's first element (three columns under a filter of five or more, whose
        // second source is past the left border) the load starts there and column 0 <- e0
        s.off = src > 0 ? src - 1 : 0;
        s.sel_lo = src > 0 ? SEL_HI : SEL_LO;
    }
    return s;
}

// Mode 2: each column on its own, one two-byte load each.
__host__ __device__ __forceinline__ PairSource pair_two_loads(int H, int W, int pad, int stride, int plane, OutPos p0, OutPos p1, int a, int b) {
    const int ih0 = p0.oh * stride + a - pad, iw0 = p0.ow * stride + b - pad;
    const int ih1 = p1.oh * stride + a - pad, iw1 = p1.ow * stride + b - pad;
    const bool v0 = (unsigned)ih0 < (unsigned)H && (unsigned)iw0 < (unsigned)W;
    const bool v1 = (unsigned)ih1 < (unsigned)H && (unsigned)iw1 < (unsigned)W;
    const int safe = min((p0.img * H + p0.oh * stride) * W + p0.ow * stride, plane - 1);
    return PairSource{v0 ? (p0.img * H + ih0) * W + iw0 : safe, v1 ? (p1.img * H + ih1) * W + iw1 : safe,
                      v0 ? SEL_LO : SEL_ZERO, v1 ? SEL_LO : SEL_ZERO};
}

}  // namespace crisp
