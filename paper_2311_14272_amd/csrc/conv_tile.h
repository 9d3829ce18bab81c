// Hybrid-sparse convolution from an input window in LDS: any filter of up to 31 taps, any stride, any width.
//
// conv_lds.h stages a patch of whole output rows with its halo, 64 channels at a time, for waves of 64 rows x 64
// columns; each wave builds the matrix core's weight operand of a kept block for 64 output positions.  Here
//   * a tile is a run of consecutive output positions, so no lane stays idle because of the image's width, and several
//     small images share a tile;
//   * what is staged is the run of input positions the tile touches, as it lies in memory -- no halo is written; a tap
//     outside the image is a bit of the lane's mask, and the lane then reads a row of zeros;
//   * as many channels are staged at once as LDS holds (usually all), so that a wave walks its whole block list between
//     two barriers;
//   * a wave owns 64 rows x 128 columns where that still fills the chip: the weight operand, which is what the vector
//     units are busy with, is built half as often.
// LDS layout: row of CC channels (+ 16 bytes) per input position, even positions first, then the odd ones.  A lane owns
// two neighbouring output columns (dword stores); at stride 1 the lanes' positions for one of the two are then
// neighbouring rows, an odd number of 16-byte units apart: conflict-free 16-byte reads (4.3 clocks per wave and
// request against 8.5 with positions in order, measured).  At stride 2 they are every second row: half of the banks, two ways.
#pragma once
#include "conv_tile_plan.h"
#include "spmm_reg.h"
#include <atomic>

namespace crisp {

constexpr uint32_t CONV_TILE_IDLE = 0x80000000u;

__device__ __forceinline__ int divide(int n, DivBy d) { return d.m ? (int)(__umulhi((uint32_t)n, d.m) >> d.shift) : n; }

// SPAN: channel counts that are no multiple of the block edge (but of eight): a block column holds K-rows of several taps.
// Every octet of K-rows is still eight channels of one tap; a table in LDS says where it lies in the chunk (or that it is
// not there: zeros), and each 16-deep step forms its own addresses from it.  A block is walked in every chunk it has a
// part in.
// APART: infinite activations at kept columns meet their weights alone (smf_apart), as the ragged product over X has it where
// a planned X gives way; with whole blocks per tap only an odd or half-even number of columns asks for that (256 x 2304 x
// 50176 2:8: 38.6 us without, 40.1 with).
template <int N, int M, int B, int NC2, bool SMF, bool SPAN, bool APART>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(conv_tile_waves(N, M, B, NC2) / 4, NC2 == 2 ? 2 : 4)))
void conv_tile_kernel(SpmmArgs p, ConvTileSched sc) {
    typedef Fmt<N, M, B> F;
    constexpr int RT = F::RT, KS = F::KS, NACC = 2 * NC2;
    typedef BlockBody<N, M, B, 1, false, 0, SMF> Body;
    // packed slices in flight per wave (ring): two where a slice is ten or twelve registers
    constexpr int R = SMF ? 2 : 1;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];     // rows, zeros, block lists, ends of runs
    constexpr bool LUT48 = lut48_pattern<N, M, SMF>();
    __shared__ u32x4 lut48[LUT48 ? 256 : 1];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nwaves = sc.RG * sc.PT;
    const int jj = lane & 31, hh = lane >> 5;
    const int r_in = wave % sc.RG, part = wave / sc.RG;
    // all block-row groups of a tile get ids on the same XCD
    const int id = blockIdx.x;
    const int xcd = id & 7, slot = id >> 3;
    const int rg = slot % sc.row_groups;
    const int tile = (slot / sc.row_groups) * 8 + xcd;
    if (tile >= sc.tiles) return;                 // the whole workgroup, before any barrier (as below)
    const int bi = rg * sc.RG + r_in;

    // ---- the tile's columns and input window --------------------------------------------------------------
    const int un = divide(tile, sc.by_unit);
    const int col_first = un * sc.unit + (tile - un * sc.per_unit) * sc.TC;
    const int col_end = min(min(col_first + sc.TC, (un + 1) * sc.unit), (int)p.Ncol);
    if (col_first >= col_end) return;
    int lo, npos;
    {
        const int row0 = divide(col_first, sc.by_Wo), row1 = divide(col_end - 1, sc.by_Wo);
        conv_tile_window_of(p.H, p.W, sc.kh, p.stride, p.pad, p.Ho, row0, row1, divide(row0, sc.by_Ho), divide(row1, sc.by_Ho), &lo, &npos);
    }
    const int zero_row = 2 * sc.HP * sc.pitch;
    uint32_t* lists = reinterpret_cast<uint32_t*>(lds + zero_row + 128);
    uint32_t* list = lists + r_in * sc.list_cap * 2;
    int* run_end = reinterpret_cast<int*>(lists + sc.RG * sc.list_cap * 2) + r_in * sc.chunks;
    // SPAN: octet of K-rows -> byte offset of its place | tap << 20 | odd shift << 30 (tap 31, which no lane has: elsewhere)
    uint32_t* octets = lists + sc.RG * (sc.list_cap * 2 + sc.chunks);

    // ---- staging: a unit is 16 channels x 128 positions; a lane takes four neighbouring positions of eight channels
    // (its half of the sixteen), 8 bytes per request, transposes them with v_perm_b32 and writes the eight channels of
    // each position with one 16-byte write.  The last lane of the window starts four positions before its end. --------
    const int pieces = (npos + 127) >> 7;
    const uint32_t pieces_inv = (65536u + (uint32_t)pieces - 1u) / (uint32_t)pieces;
    auto units_of = [&](int q) __attribute__((always_inline)) { return ((min(sc.CC, p.C - q * sc.CC) + (SPAN ? 8 : 0)) >> 4) * pieces; };
    auto request = [&](int q, int u, u32x2 (&v)[8]) __attribute__((always_inline)) {
        const uint32_t plane_bytes = (uint32_t)p.plane * 2u;
        u = min(u, units_of(q) - 1);
        const int g = (int)(((uint32_t)u * pieces_inv) >> 16), pc = u - g * pieces;
        const rsrc_t r = make_rsrc(p.act + (int64_t)(q * sc.CC + g * 16) * p.plane + lo);
        // (SPAN: an odd number of octets leaves the upper half of the last unit without channels: it re-reads the lower's)
        const uint32_t upper = SPAN && q * sc.CC + g * 16 + 8 >= p.C ? 0u : (uint32_t)hh;
        const uint32_t off = upper * 8u * plane_bytes + (uint32_t)min(pc * 128 + jj * 4, npos - 4) * 2u;
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = buf_load_x<2>(r, off, (uint32_t)i * plane_bytes);
    };
    auto deposit = [&](int q, int u, const u32x2 (&v)[8]) __attribute__((always_inline)) {
        if (u >= units_of(q)) return;
        const int g = (int)(((uint32_t)u * pieces_inv) >> 16), pc = u - g * pieces;
        if (pc * 128 + jj * 4 >= npos || (SPAN && q * sc.CC + g * 16 + hh * 8 >= p.C)) return;
        const int first = min(pc * 128 + jj * 4, npos - 4);
        const uint32_t at = (uint32_t)((g * 16 + hh * 8) * 2);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            u32x4 o;
#pragma unroll
            for (int x = 0; x < 4; ++x)
                o[x] = __builtin_amdgcn_perm(v[2 * x + 1][j >> 1], v[2 * x][j >> 1], (j & 1) ? SEL_HI : SEL_LO);
            const int pos = first + j;
            *reinterpret_cast<u32x4*>(lds + (uint32_t)(((pos & 1) * sc.HP + (pos >> 1)) * sc.pitch) + at) = o;
        }
    };
    auto stage = [&](int q, int u0) __attribute__((always_inline)) {
        constexpr int UN = 2;
        for (; u0 < units_of(q); u0 += nwaves * UN) {
            u32x2 v[UN][8];
#pragma unroll
            for (int k = 0; k < UN; ++k) request(q, u0 + k * nwaves, v[k]);
#pragma unroll
            for (int k = 0; k < UN; ++k) deposit(q, u0 + k * nwaves, v[k]);
        }
    };
    // the first units are requested before anything else; the lists and the lanes' addresses are formed meanwhile
    constexpr int UN0 = 4;
    u32x2 ahead[UN0][8];
#pragma unroll
    for (int k = 0; k < UN0; ++k) request(0, wave + k * nwaves, ahead[k]);
    __builtin_amdgcn_sched_barrier(0);

    // ---- lane constants: for each of its columns the place of the filter's first tap (for an even and an odd shift
    // of the position) and the taps inside the image; columns past the tile have none -----------------------------
    uint32_t base_even[NACC], base_odd[NACC], inside[NACC];
    const int part_col = col_first + part * 64 * NC2;
#pragma unroll
    for (int c2 = 0; c2 < NC2; ++c2) {
        const int n0 = part_col + c2 * 64 + 2 * jj;
        const int j = n0 < col_end ? n0 : col_first;
        const int row = divide(j, sc.by_Wo);
        int ow = j - row * p.Wo, img = divide(row, sc.by_Ho), oh = row - img * p.Ho;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            if (c == 1) {
                if (++ow == p.Wo) { ow = 0; ++oh; }
                if (oh == p.Ho) { oh = 0; ++img; }
            }
            const int ih = oh * p.stride - p.pad, iw = ow * p.stride - p.pad;
            const int pos = (img * p.H + ih) * p.W + iw - lo;
            base_even[2 * c2 + c] = (uint32_t)(((pos & 1) * sc.HP + (pos >> 1)) * sc.pitch + (SPAN ? 0 : hh * 16));
            base_odd[2 * c2 + c] = (uint32_t)((((pos + 1) & 1) * sc.HP + ((pos + 1) >> 1)) * sc.pitch + (SPAN ? 0 : hh * 16));
            uint32_t cols_in = 0, taps_in = 0;
            for (int b = 0; b < p.kw; ++b) cols_in |= ((unsigned)(iw + b) < (unsigned)p.W ? 1u : 0u) << b;
            for (int a = 0; a < sc.kh; ++a) taps_in |= ((unsigned)(ih + a) < (unsigned)p.H ? cols_in : 0u) << (a * p.kw);
            inside[2 * c2 + c] = n0 + c < col_end ? taps_in : 0u;
        }
    }
    const bool works = bi < p.Sb && col_first + part * 64 * NC2 < col_end;
    int t_begin = 0, cnt = 0;
    if (bi < p.Sb) {
        t_begin = p.row_ptr[bi];
        cnt = p.row_ptr[bi + 1] - t_begin;
    }
    const bool busy = works && cnt > 0;
    const uint32_t a_off = (uint32_t)((jj * F::SLOTS + hh * F::FS * (SMF ? 2 : 1)) * 2);
    const uint32_t i_off = (uint32_t)(jj * F::WPR * 4);
    const uint32_t aw_sh = (uint32_t)hh * F::HB * (SMF ? 2 : 1);
    uint32_t av[R][RT][KS][F::VW], aw[R][RT][F::WPR];
    // one chunk: the list is the packed order, and the first slices can be requested at once
    if (busy && sc.chunks == 1) {
#pragma unroll
        for (int r = 0; r < R; ++r) Body::load_a(av[r], aw[r], p, a_off, i_off, t_begin + min(r, cnt - 1));
    }
    // ---- block lists: one wave per block-row; entry: block (from the row's first) | tap << 16 | odd shift << 24,
    // byte offset of the tap and channel block inside the staged chunk -----------------------------------------
    if (part == 0) {
        int place = 0;
        const float inv_CB = 1.0f / (float)sc.CB, inv_CBC = 1.0f / (float)sc.CBC;
        for (int q = 0; q < sc.chunks; ++q) {
            for (int e0 = 0; e0 < cnt; e0 += 64) {
                const int e = e0 + lane;
                const int bj = p.col_idx[t_begin + min(e, cnt - 1)];
                const int tap = (int)(((float)bj + 0.5f) * inv_CB), cb = bj - tap * sc.CB;
                bool here = e < cnt;
                if constexpr (SPAN) {              // any octet of the block's rows with channels of this chunk
                    bool any = sc.chunks == 1;
                    for (int o = 0; o < B / 8 && !__all(any); ++o) {
                        const int k = bj * B + o * 8, c = k - (int)(((float)k + 0.5f) * p.inv_C) * p.C;
                        any = any || (k < p.K && c >= q * sc.CC && c < (q + 1) * sc.CC);
                    }
                    here = here && any;
                } else {
                    here = here && (int)(((float)cb + 0.5f) * inv_CBC) == q;
                }
                const unsigned long long ballot = __ballot(here);
                if (here) {
                    const int a = (int)(((float)tap + 0.5f) * p.inv_kw), b = tap - a * p.kw;
                    const int shift = a * p.W + b;
                    const int at = place + __popcll(ballot & ((1ull << lane) - 1ull));
                    list[2 * at] = SPAN ? (uint32_t)e : (uint32_t)e | (uint32_t)tap << 16 | (uint32_t)(shift & 1) << 24;
                    list[2 * at + 1] = SPAN ? (uint32_t)(bj * (B / 8)) : (uint32_t)((shift >> 1) * sc.pitch + (cb - q * sc.CBC) * (B * 2));
                }
                place += __popcll(ballot);
            }
            if (R == 2 && (place & 1)) {           // runs of whole ring turns
                if (lane == 0) { list[2 * place] = CONV_TILE_IDLE; list[2 * place + 1] = 0u; }
                ++place;
            }
            if (lane == 0) run_end[q] = place;
        }
        if (lane < R) { list[2 * (place + lane)] = CONV_TILE_IDLE; list[2 * (place + lane) + 1] = 0u; }
    }
    auto fill_octets = [&](int q) __attribute__((always_inline)) {
        for (int o = tid; o < sc.octets; o += 64 * nwaves) {
            const int k = o * 8, tap = (int)(((float)k + 0.5f) * p.inv_C), c = k - tap * p.C - q * sc.CC;
            const int a = (int)(((float)tap + 0.5f) * p.inv_kw), b = tap - a * p.kw;
            const int shift = a * p.W + b;
            octets[o] = k < p.K && c >= 0 && c < sc.CC
                ? (uint32_t)((shift >> 1) * sc.pitch + c * 2) | (uint32_t)tap << 20 | (uint32_t)(shift & 1) << 30 : 31u << 20;
        }
    };
    if constexpr (SPAN) fill_octets(0);
    if (tid < 8) reinterpret_cast<u32x4*>(lds + zero_row)[tid] = u32x4{0u, 0u, 0u, 0u};
    if constexpr (LUT48) lut48_fill(lut48, tid, 64 * nwaves);


    // ---- first chunk into LDS --------------------------------------------------------------------------------
#pragma unroll
    for (int k = 0; k < UN0; ++k) deposit(0, wave + k * nwaves, ahead[k]);
    stage(0, wave + UN0 * nwaves);

    f32x16 acc[RT][NACC];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int c = 0; c < NACC; ++c)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[rt][c][r] = 0.0f;

    // one kept block
    auto multiply = [&](uint32_t (&av)[RT][KS][F::VW], const uint32_t (&aw)[RT][F::WPR], uint32_t what, uint32_t off) __attribute__((always_inline)) {
        uint32_t ws[RT][F::WPR];
        if constexpr (N != M) {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int i = 0; i < F::WPR; ++i)
                    ws[rt][i] = __builtin_amdgcn_alignbit(i + 1 < F::WPR ? aw[rt][i + 1] : 0u, aw[rt][i], aw_sh);
        }
        // the eight K-rows of the lane's half of 16-deep step ks, at its columns
        const unsigned char* base[NACC];
        if constexpr (!SPAN) {
            const int tap = (int)(what >> 16) & 31;
            const bool odd = (what >> 24) & 1u;
#pragma unroll
            for (int c = 0; c < NACC; ++c) {
                const uint32_t in = (uint32_t)__builtin_amdgcn_sbfe((int)inside[c], tap, 1);
                const uint32_t at = (odd ? base_odd[c] : base_even[c]) + off;
                base[c] = lds + ((at & in) | ((uint32_t)zero_row & ~in));
            }
        }
        uint32_t oct[SPAN ? KS : 1];
        if constexpr (SPAN) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) oct[ks] = octets[off + ks * 2 + hh];
            // Several chunks: weights whose K-rows are not in this one count in another.  They are cleared here, as an
            // infinite one times the zeros that stand for its rows would be NaN.  (A lane's values av[..][ks] belong to octet
            // 2 ks + hh, as sparse operands to the two neighbouring octets of its sixteen columns.  Once per block on the
            // packed values: as part of each operand it cost 1.5 % of every case, one chunk or more.)
            if (sc.chunks > 1) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    const uint32_t o = SMF ? octets[off + (ks & ~1) * 2 + hh * 2 + (ks & 1)] : oct[ks];
                    const uint32_t here = (o >> 20 & 31u) == 31u ? 0u : 0xFFFFFFFFu;
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                        for (int x = 0; x < F::VW; ++x) av[rt][ks][x] &= here;
                }
            }
        }
        auto rows_at = [&](int c, int ks) __attribute__((always_inline)) {
            if constexpr (SPAN) {
                const uint32_t in = (uint32_t)((int)(inside[c] << (31u - (oct[ks] >> 20 & 31u))) >> 31);
                const uint32_t at = ((oct[ks] >> 30) ? base_odd[c] : base_even[c]) + (oct[ks] & 0xFFFFFu);
                return *reinterpret_cast<const u32x4*>(lds + ((at & in) | ((uint32_t)zero_row & ~in)));
            } else {
                return *reinterpret_cast<const u32x4*>(base[c] + ks * 32);
            }
        };
        if constexpr (SMF) {
            typedef __attribute__((ext_vector_type(8))) uint32_t u32x8;
            auto sparse_step = [&](auto s2_c) __attribute__((always_inline)) {
                constexpr int s2 = decltype(s2_c)::value;
                u32x8 b8[NACC];
#pragma unroll
                for (int c = 0; c < NACC; ++c) {
                    const u32x4 l4 = rows_at(c, 2 * s2);
                    const u32x4 h4 = rows_at(c, 2 * s2 + 1);
                    b8[c] = u32x8{l4[0], l4[1], l4[2], l4[3], h4[0], h4[1], h4[2], h4[3]};
                }
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) {
                    u32x4 a4;
                    uint32_t idx;
                    smf_operand<N, M, B, s2>(av[rt], ws[rt], a4, idx);
                    if constexpr (APART) idx = smf_apart<N, M>(idx);
                    const bf16x8 afrag = __builtin_bit_cast(bf16x8, a4);
#pragma unroll
                    for (int c = 0; c < NACC; ++c)
                        acc[rt][c] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(afrag, __builtin_bit_cast(bf16x16, b8[c]), acc[rt][c],
                                                                               (int)idx, 0, 0);
                }
            };
            sparse_step(std::integral_constant<int, 0>{});
            if constexpr (KS == 4) sparse_step(std::integral_constant<int, 1>{});
        } else {
            auto dense_step = [&](auto ks_c) __attribute__((always_inline)) {
                constexpr int ks = decltype(ks_c)::value;
                bf16x8 bfrag[NACC];
#pragma unroll
                for (int c = 0; c < NACC; ++c) bfrag[c] = __builtin_bit_cast(bf16x8, rows_at(c, ks));
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) {
                    u32x4 a4;
                    if constexpr (LUT48) a4 = expand_frag_lut48<B, ks>(av[rt][ks], ws[rt], lut48);
                    else a4 = expand_frag<N, M, B, ks>(av[rt][ks], ws[rt]);
                    const bf16x8 afrag = __builtin_bit_cast(bf16x8, a4);
#pragma unroll
                    for (int c = 0; c < NACC; ++c)
                        acc[rt][c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(afrag, bfrag[c], acc[rt][c], 0, 0, 0);
                }
            };
            dense_step(std::integral_constant<int, 0>{});
            dense_step(std::integral_constant<int, 1>{});
            if constexpr (KS == 4) {
                dense_step(std::integral_constant<int, 2>{});
                dense_step(std::integral_constant<int, 3>{});
            }
        }
    };

    int e = 0;
    for (int q = 0; q < sc.chunks; ++q) {
        if (q > 0) {
            __syncthreads();                       // everybody is done with the previous chunk
            if constexpr (SPAN) fill_octets(q);
            stage(q, wave);
        }
        __syncthreads();
        if (busy) {
            auto entry = [&](int i, uint32_t& what, uint32_t& off) __attribute__((always_inline)) {
                what = (uint32_t)__builtin_amdgcn_readfirstlane((int)list[2 * i]);
                off = (uint32_t)__builtin_amdgcn_readfirstlane((int)list[2 * i + 1]);
            };
            const int e_end = __builtin_amdgcn_readfirstlane(run_end[q]);
            uint32_t what[R], off[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                entry(e + r, what[r], off[r]);
                if (q == 0 && sc.chunks > 1) Body::load_a(av[r], aw[r], p, a_off, i_off, t_begin + (int)(what[r] & 0xFFFFu));
            }
            for (; e < e_end; e += R) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    uint32_t what_next, off_next;
                    entry(e + r + R, what_next, off_next);
                    // the slice must have arrived whether or not the entry is idle (wait outside the branch)
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt) {
#pragma unroll
                        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                            for (int x = 0; x < F::VW; ++x) asm volatile("" ::"v"(av[r][rt][ks][x]));
                        if constexpr (N != M) {
#pragma unroll
                            for (int x = 0; x < F::WPR; ++x) asm volatile("" ::"v"(aw[r][rt][x]));
                        }
                    }
                    if (!(what[r] & CONV_TILE_IDLE)) multiply(av[r], aw[r], what[r], off[r]);
                    Body::load_a(av[r], aw[r], p, a_off, i_off, t_begin + (int)(what_next & 0xFFFFu));   // past the end: an idle entry
                    what[r] = what_next;
                    off[r] = off_next;
                }
            }
        }
    }
    if (works) {
        // (row addresses from an opaque copy of the lane's row half: not all formed beforehand and spilled)
        int hh_now = hh;
        asm volatile("" : "+v"(hh_now));
#pragma unroll
        for (int c2 = 0; c2 < NC2; ++c2) {
            const int64_t col0 = part_col + c2 * 64 + 2 * jj;
#pragma unroll
            for (int r0 = 0; r0 < RT * 16; r0 += 16)
                store_rows<B, 1, 16, 1>(p, bi, hh_now, col0, col0 + 1 < col_end, r0, [&](int pr, float (&v)[2]) __attribute__((always_inline)) {
#pragma unroll
                    for (int c = 0; c < 2; ++c) v[c] = acc[pr >> 4][2 * c2 + c][pr & 15];
                });
        }
        // An odd number of columns in all: the last one, a row per lane, out of the two lanes that hold it.  With the
        // column left to store_rows every case pays: 256 x 2304 x 50176 2:8 37.8 us, 39.6 with its question at each row,
        // 39.3 and spilled registers with a second copy of the stores.
        const int last = col_end - 1 - part_col;
        if ((col_end & 1) && last < 64 * NC2) {
            const int from = (last & 63) >> 1;
            float mine[1] = {0.0f};
#pragma unroll
            for (int c2 = 0; c2 < NC2; ++c2) {
                if (last >> 6 != c2) continue;
#pragma unroll
                for (int pr = 0; pr < RT * 16; ++pr) {
                    const int row = (pr >> 4) * 32 + 8 * ((pr & 15) >> 2) + (pr & 3);
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const uint32_t v = __builtin_amdgcn_readlane(__float_as_uint(acc[pr >> 4][2 * c2][pr & 15]), from + 32 * h);
                        mine[0] = lane == row + 4 * h ? __uint_as_float(v) : mine[0];
                    }
                }
            }
            const int row = bi * B + lane;
            if (lane < B && row < p.S) {
                apply_epilogue<1>(p, row, col_end - 1, true, mine);
                const int64_t at = (int64_t)row * p.ldy + col_end - 1;
                if (p.y_bf16) {
                    const f32x2 two = {mine[0], mine[0]};
                    reinterpret_cast<uint16_t*>(p.Y)[at] = (uint16_t)__builtin_bit_cast(uint32_t, __builtin_convertvector(two, bf16x2));
                } else {
                    reinterpret_cast<float*>(p.Y)[at] = mine[0];
                }
            }
        }
    }
}

template <int N, int M, int B, int NC2, bool SMF, bool SPAN, bool APART>
hipError_t launch_conv_tile_k(const SpmmArgs& a, const ConvTileSched& s, hipStream_t st) {
    const int64_t wgs = (int64_t)((s.tiles + 7) / 8) * 8 * s.row_groups;
    if (wgs > INT32_MAX) return hipErrorInvalidValue;
    if (s.lds_bytes > 60 * 1024) {
        // more dynamic LDS than a kernel gets by default: raised once per device for this instantiation
        static std::atomic<uint64_t> raised{0};
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
        if (!(raised.load() >> dev & 1)) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&conv_tile_kernel<N, M, B, NC2, SMF, SPAN, APART>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, CONV_TILE_MAX_LDS);
            if (e != hipSuccess) return e;
            raised.fetch_or((uint64_t)1 << dev);
        }
    }
    const dim3 grd((unsigned)wgs), blk(64 * s.RG * s.PT);
    if (a.ev_start || a.ev_stop)
        hipExtLaunchKernelGGL((conv_tile_kernel<N, M, B, NC2, SMF, SPAN, APART>), grd, blk, (size_t)s.lds_bytes, st, a.ev_start, a.ev_stop, 0, a, s);
    else
        conv_tile_kernel<N, M, B, NC2, SMF, SPAN, APART><<<grd, blk, (size_t)s.lds_bytes, st>>>(a, s);
    return hipGetLastError();
}

template <int N, int M, int B, bool SPAN>
hipError_t launch_conv_tile_b(const SpmmArgs& a, const ConvTileSched& s, hipStream_t st) {
    constexpr bool SMF = smf_pattern<N, M>();
    if constexpr (SMF && !SPAN) {
        if ((a.Ncol & 3) == 0)
            return s.NC2 == 2 ? launch_conv_tile_k<N, M, B, 2, SMF, SPAN, false>(a, s, st)
                              : launch_conv_tile_k<N, M, B, 1, SMF, SPAN, false>(a, s, st);
    }
    return s.NC2 == 2 ? launch_conv_tile_k<N, M, B, 2, SMF, SPAN, SMF>(a, s, st) : launch_conv_tile_k<N, M, B, 1, SMF, SPAN, SMF>(a, s, st);
}

template <int N, int M>
hipError_t launch_conv_tile(const SpmmArgs& a, int B, const ConvTileSched& s, hipStream_t st) {
    if (s.octets) return B == 64 ? launch_conv_tile_b<N, M, 64, true>(a, s, st) : launch_conv_tile_b<N, M, 32, true>(a, s, st);
    return B == 64 ? launch_conv_tile_b<N, M, 64, false>(a, s, st) : launch_conv_tile_b<N, M, 32, false>(a, s, st);
}

}  // namespace crisp
