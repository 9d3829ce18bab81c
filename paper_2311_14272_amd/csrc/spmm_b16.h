// Hybrid-sparse product with 16 x 16 blocks (the paper's smallest block size), for the patterns with a kernel of their own.
//
// Two kept blocks of a block-row, wherever they lie, are one v_mfma_f32_16x16x32_bf16: lane (j = lane % 16, q = lane / 16)
// supplies row j of block q / 2, columns 8 (q % 2) .. + 7, and for its eight output columns the eight K-rows behind them, so
// neither operand is ever half empty.  A wave owns one block-row and a strip of 128 columns: a lane's eight columns are one
// 16-byte request per K-row, the packed slice is expanded once for eight matrix-core instructions, and rows of Y leave in
// 16-byte stores.  PF pairs of blocks are on their way while one is multiplied; block numbers are scalar.
//   NWK == 1: the four waves of a workgroup take four neighbouring block-rows of one strip, whose X rows they find in the
//             level-1 cache;
//   NWK == 4: they split one block-row's list (few tiles), partial sums added in a fixed order through LDS.
// Bound by the requests for X (4 KB per kept block and 128 columns) and, on few tiles, by latency.  Against one block
// at a time without anything requested ahead, 64 columns per wave (before / now): 64 x 2144 x 125200 3:4 241 / 147 us (2.9 / 4.8
// TB/s), 64 x 3840 x 1173 1:4 88 / 10.5 us, 1408 x 4416 x 5520 4:8 618 / 162 us.
#pragma once
#include "packed_addr.h"
#include "spmm_reg.h"

namespace crisp {

typedef __attribute__((ext_vector_type(4))) float f32x4v;

template <int N, int M, int NWK, bool RAGGED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 3)))
void spmm_b16_pair_kernel(SpmmArgs p) {
    typedef Fmt<N, M, 16> F;
    constexpr int PF = 2;                         // pairs in flight
    const int id = blockIdx.x;
    const int xcd = id & 7, slot = id >> 3;
    const int row_groups = NWK == 1 ? (p.Sb + 3) / 4 : p.Sb;
    const int rg = slot % row_groups;
    const int nt = (slot / row_groups) * 8 + xcd;
    if (nt >= p.NT) return;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int bi = NWK == 1 ? rg * 4 + wave : rg;
    constexpr bool LUT48 = lut48_pattern<N, M, false>();
    __shared__ u32x4 lut48[LUT48 ? 256 : 1];
    if constexpr (LUT48) {
        lut48_fill(lut48, threadIdx.x, 256);
        __syncthreads();
    }
    if (NWK == 1 && bi >= p.Sb) return;           // no further barriers in this mode
    const int j = lane & 15, q = lane >> 4, second = q >> 1, half = q & 1;
    const int64_t col0 = (int64_t)nt * 128 + j * 8;
    const bool col_ok = col0 < p.Ncol;            // ldx % 8 == 0: the lane's 16 bytes stay in the row
    const uint16_t* xlane = p.X + (col_ok ? col0 : 0);
    const int t_begin = p.row_ptr[bi], t_end = p.row_ptr[bi + 1];
    const int pairs = (t_end - t_begin + 1) / 2;
    const int first = NWK == 1 ? 0 : wave;
    const int cnt = first < pairs ? (pairs - first + NWK - 1) / NWK : 0;

    f32x4v acc[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[c] = f32x4v{0.f, 0.f, 0.f, 0.f};
    u32x4 xr[PF][8];
    uint32_t av[PF][F::VW], aw[PF][F::WPR];
    bool there[PF];                               // the lane's block of the pair exists

    auto request = [&](int d, int pair) __attribute__((always_inline)) {
        const int t0 = t_begin + 2 * pair, t1 = min(t0 + 1, t_end - 1);
        const int bj0 = p.col_idx[t0], bj1 = p.col_idx[t1];
        const int t = second ? t1 : t0, kb = (second ? bj1 : bj0) * 16 + half * 8;
        there[d] = !second || t0 + 1 < t_end;
        const uint16_t* src = xlane + (int64_t)kb * p.ldx;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if constexpr (RAGGED) {
                // rows at or past K re-read the last one and are zeroed when used
                xr[d][i] = *reinterpret_cast<const u32x4*>(xlane + (int64_t)min(kb + i, p.K - 1) * p.ldx);
                if (kb + i >= p.K) xr[d][i] = u32x4{0u, 0u, 0u, 0u};
            } else {
                xr[d][i] = *reinterpret_cast<const u32x4*>(src + (int64_t)i * p.ldx);
            }
        }
        const rsrc_t rv = make_rsrc(p.vals), ri = make_rsrc(p.idxw);
        load_vals<F::FS>(rv, b16_value_at(t, j, F::SLOTS, half * F::FS), 0, av[d]);
        if constexpr (N != M) load_positions<F::WPR>(ri, b16_words_at(t, j, F::WPR), 0, aw[d]);
    };
    auto multiply = [&](int d) __attribute__((always_inline)) {
        // a list of odd length: the last pair's second block is zero in both operands (an infinite element of X times a
        // zero weight would not be)
        u32x4 a4;
        uint32_t ws[F::WPR];
        if constexpr (N != M) {
#pragma unroll
            for (int i = 0; i < F::WPR; ++i)
                ws[i] = __builtin_amdgcn_alignbit(i + 1 < F::WPR ? aw[d][i + 1] : 0u, aw[d][i], (uint32_t)(half * F::HB));
        }
        if constexpr (LUT48) a4 = expand_frag_lut48<16, 0>(av[d], ws, lut48);
        else a4 = expand_frag<N, M, 16, 0>(av[d], ws);
        const uint32_t keep = there[d] ? 0xFFFFFFFFu : 0u;
        a4 = a4 & u32x4{keep, keep, keep, keep};
        const bf16x8 afrag = __builtin_bit_cast(bf16x8, a4);
        const uint32_t lo = there[d] ? SEL_LO : SEL_ZERO, hi = there[d] ? SEL_HI : SEL_ZERO;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            u32x4 b4;
#pragma unroll
            for (int x = 0; x < 4; ++x) b4[x] = __builtin_amdgcn_perm(xr[d][2 * x + 1][c >> 1], xr[d][2 * x][c >> 1], (c & 1) ? hi : lo);
            acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(afrag, __builtin_bit_cast(bf16x8, b4), acc[c], 0, 0, 0);
        }
    };
#pragma unroll
    for (int d = 0; d < PF; ++d)
        if (d < cnt) request(d, first + d * NWK);
    int i = 0;
    for (; i + 2 * PF <= cnt; i += PF) {
#pragma unroll
        for (int d = 0; d < PF; ++d) {
            multiply(d);
            request(d, first + (i + d + PF) * NWK);
        }
    }
#pragma unroll
    for (int e = 0; e < 2 * PF - 1; ++e) {
        if (i + e < cnt) {
            multiply(e % PF);
            if (e < PF - 1 && i + e + PF < cnt) request(e % PF, first + (i + e + PF) * NWK);
        }
    }

    // ---- rows 4q .. 4q + 3 of the block-row, columns col0 .. col0 + 7 -------------------------------------------
    int row_first = 0;
    if constexpr (NWK > 1) {
        __shared__ f32x4v red[NWK][8][64];
#pragma unroll
        for (int c = 0; c < 8; ++c) red[wave][c][lane] = acc[c];
        __syncthreads();
        // wave w adds up and stores row 4q + w
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            float s = red[0][c][lane][wave];
#pragma unroll
            for (int w = 1; w < NWK; ++w) s += red[w][c][lane][wave];
            acc[c][0] = s;
        }
        row_first = wave;
    }
    if (!col_ok) return;
    const bool full = col0 + 8 <= p.Ncol;
    constexpr int ROWS = NWK > 1 ? 1 : 4;
    const int row0 = bi * 16 + 4 * q + row_first;
    // The epilogue of all values before the first store, its operands requested together: with a branch or a store between
    // them every one waits out a trip to memory (80 x 64 x 167 2:8 with scale, bias and ReLU, whose rows end inside a lane:
    // 11.6 us one by one, 6.7 so).
    float v[ROWS][8];
#pragma unroll
    for (int r = 0; r < ROWS; ++r)
#pragma unroll
        for (int c = 0; c < 8; ++c) v[r][c] = acc[c][r];
    if (p.ep_on) {
        float sc[ROWS] = {}, bs[ROWS] = {};
        int rows[ROWS];
#pragma unroll
        for (int r = 0; r < ROWS; ++r) rows[r] = min(row0 + r, p.S - 1);
        if (p.ep_scale)
#pragma unroll
            for (int r = 0; r < ROWS; ++r) sc[r] = p.ep_scale[rows[r]];
        if (p.ep_bias)
#pragma unroll
            for (int r = 0; r < ROWS; ++r) bs[r] = p.ep_bias[rows[r]];
        const int left = (int)min(p.Ncol - col0, (int64_t)8) - 1;      // the lane's last column that exists
        if (p.y_bf16) {
            uint32_t res[ROWS][4] = {};
            const uint16_t* src = reinterpret_cast<const uint16_t*>(p.ep_res) + col0;
            if (p.ep_res && full) {
#pragma unroll
                for (int r = 0; r < ROWS; ++r) {
                    const u32x4 t = *reinterpret_cast<const u32x4*>(src + (int64_t)rows[r] * p.ep_ldr);
#pragma unroll
                    for (int x = 0; x < 4; ++x) res[r][x] = t[x];
                }
            } else if (p.ep_res) {
#pragma unroll
                for (int r = 0; r < ROWS; ++r)
#pragma unroll
                    for (int c = 0; c < 8; ++c) res[r][c >> 1] |= (uint32_t)src[(int64_t)rows[r] * p.ep_ldr + min(c, left)] << 16 * (c & 1);
            }
#pragma unroll
            for (int r = 0; r < ROWS; ++r) ep_apply<8, true>(p, res[r], sc[r], bs[r], v[r]);
        } else {
            uint32_t res[ROWS][8] = {};
            const uint32_t* src = reinterpret_cast<const uint32_t*>(p.ep_res) + col0;
            if (p.ep_res && full) {
#pragma unroll
                for (int r = 0; r < ROWS; ++r)
#pragma unroll
                    for (int c = 0; c < 8; ++c) res[r][c] = src[(int64_t)rows[r] * p.ep_ldr + c];
            } else if (p.ep_res) {
#pragma unroll
                for (int r = 0; r < ROWS; ++r)
#pragma unroll
                    for (int c = 0; c < 8; ++c) res[r][c] = src[(int64_t)rows[r] * p.ep_ldr + min(c, left)];
            }
#pragma unroll
            for (int r = 0; r < ROWS; ++r) ep_apply<8, false>(p, res[r], sc[r], bs[r], v[r]);
        }
    }
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const int row = row0 + r;
        if (row >= p.S) continue;
        if (full) {
            if (p.y_bf16) {
                u32x4 pk;
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const f32x2 two = {v[r][2 * x], v[r][2 * x + 1]};
                    pk[x] = __builtin_bit_cast(uint32_t, __builtin_convertvector(two, bf16x2));
                }
                *reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(p.Y) + (int64_t)row * p.ldy + col0) = pk;
            } else {
                float* y = reinterpret_cast<float*>(p.Y) + (int64_t)row * p.ldy + col0;
                *reinterpret_cast<float4*>(y) = make_float4(v[r][0], v[r][1], v[r][2], v[r][3]);
                *reinterpret_cast<float4*>(y + 4) = make_float4(v[r][4], v[r][5], v[r][6], v[r][7]);
            }
        } else {
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                if (col0 + c >= p.Ncol) continue;
                const float one = v[r][c];
                if (p.y_bf16) reinterpret_cast<uint16_t*>(p.Y)[(int64_t)row * p.ldy + col0 + c] = float_to_bf16_rne(one);
                else reinterpret_cast<float*>(p.Y)[(int64_t)row * p.ldy + col0 + c] = one;
            }
        }
    }
}

template <int N, int M, int NWK, bool RAGGED>
hipError_t launch_b16_k(const SpmmArgs& a, hipStream_t st) {
    SpmmArgs p = a;
    p.NT = (int)((a.Ncol + 127) / 128);
    const int64_t groups = (int64_t)((p.NT + 7) / 8) * (NWK == 1 ? (a.Sb + 3) / 4 : a.Sb) * 8;
    if (groups > INT32_MAX) return hipErrorInvalidValue;
    if (a.ev_start || a.ev_stop)
        hipExtLaunchKernelGGL((spmm_b16_pair_kernel<N, M, NWK, RAGGED>), dim3((unsigned)groups), dim3(256), 0, st, a.ev_start, a.ev_stop, 0, p);
    else
        spmm_b16_pair_kernel<N, M, NWK, RAGGED><<<dim3((unsigned)groups), dim3(256), 0, st>>>(p);
    return hipGetLastError();
}

// split: four waves share a block-row's list
template <int N, int M>
hipError_t launch_b16(const SpmmArgs& a, bool split, hipStream_t st) {
    if (a.K % 16) return split ? launch_b16_k<N, M, 4, true>(a, st) : launch_b16_k<N, M, 1, true>(a, st);
    return split ? launch_b16_k<N, M, 4, false>(a, st) : launch_b16_k<N, M, 1, false>(a, st);
}

}  // namespace crisp
