// Mask selection kernels: saliency -> N:M choice -> block scores -> block choice.
// Alg. 1 lines 2, 4-6 and 10 of the CRISP paper; every ordering decision below is a total
// order so that the result is unique and reproducible bit for bit.
#include "select_lane.h"

namespace crisp {

// One workgroup per B x B block, Q lanes per block row (Q * CPT = B columns, CPT = 16).
// Each lane loads its CPT weights (and gradient / saliency values) with 16-byte loads, ranks
// every aligned group of M columns (keep the n first under: larger saliency first, on a tie the
// smaller column first), and leaves "saliency if kept else +0" in LDS.  The Q lanes of a row
// OR their mask bits together with xor-shuffles.  Then lane r of the first wave adds row r's B
// values left to right in fp64 and lane 0 adds the row sums top to bottom: that summation order
// is part of the definition of the block score (a tree reduction would round differently;
// adding +0.0 for a pruned element leaves the non-negative running sum unchanged bit for bit).
// PACK: while the block's weights and keep bits are in registers, its packed form (compressed
// values, position stream, 2-of-4 violation) is also written, to a staging area indexed by the
// block's place in the grid; whether the block is kept is only known after the block choice,
// which then just copies the kept blocks' packed forms to their final place (topk_gather_kernel).
// Up to CAP layers of equal (B, saliency kind) share one launch: a model's layers have block grids of a few dozen to a few
// hundred workgroups each, far too few to fill 256 compute units one layer at a time, and a launch has a ramp and a last
// wave of its own (the 53 layers of ResNet-50: two launches in place of eight, one pair per pattern width and alignment,
// 82 -> 47 us on the GPU).  Workgroup ids are mapped to (layer, block) through the prefix sums in `first`.
template <int THREADS, class LAYER, int CAP>
__device__ __forceinline__ int layer_of(const SelBatch<LAYER, CAP>& bt, int id) {
    if constexpr (CAP == 1) return 0;
    const int lane = threadIdx.x & 63;
    return layer_by_ballots<THREADS, CAP>(bt.n, bt.first, id, [&](auto p) __attribute__((always_inline)) { return __ballot(p(lane)); });
}

// Saliency, N:M choice and (PACK) packed form of one lane's columns; returns the keep bits.
template <int B, int M, int KIND, bool VEC, bool PACK>
__device__ __forceinline__ uint32_t score_lane(const ScoreLayer& sa, const SelStage& stg, size_t blk, int r, int s, int c0, int k0,
                                               float* kept_dst, uint32_t* pos_row, int wmax, int* viol) {
    constexpr bool NEEDW = PACK || KIND != CRISP_SAL_GIVEN;
    const int len = (s < sa.S) ? min(LANE_COLS, sa.K - k0) : 0;   // columns of this lane that exist (may be <= 0)
    LaneRaw raw;
    lane_load<KIND, VEC, NEEDW>(raw, sa.W, sa.TG, (size_t)min(s, sa.S - 1) * sa.K, k0, sa.K);
    const uint32_t bits = lane_select<M, KIND, NEEDW, true>(raw, sa.n, len, kept_dst);
    if constexpr (PACK) {
        // packed form of the lane's groups, to the block's staging area
        const int slot0 = (c0 / M) * sa.n;
        uint16_t* sv = reinterpret_cast<uint16_t*>(sa.stage + stg.vals_off) + (blk * B + r) * stg.slots + slot0;
        uint16_t w[LANE_COLS];
        lane_weights(raw, len, w);
        if (lane_pack<M>(w, bits, sa.n, stg.wbits, s >= sa.S, k0, sa.K, sv, pos_row, slot0, wmax)) *viol = 1;
    }
    return bits;
}

template <int B, int KIND, bool PACK, int CAP>
__global__ __launch_bounds__(score_threads(B)) void score_select_kernel(SelBatch<ScoreLayer, CAP> bt) {
    constexpr int NTHR = score_threads(B);
    const int li = __builtin_amdgcn_readfirstlane(layer_of<NTHR>(bt, (int)blockIdx.x));
    const ScoreLayer& sa = bt.L[li];
    const int local = (int)blockIdx.x - bt.first[li];
    const int S = sa.S, K = sa.K;
    const int Kb = (K + B - 1) / B, mwpr = (K + 31) / 32;
    uint32_t* __restrict__ nm_mask = sa.nm_mask;
    const SelStage stg = sel_stage(B, sa.n, sa.m, (size_t)((S + B - 1) / B) * Kb);
    constexpr int Q = B / LANE_COLS;  // lanes per block row (1, 2 or 4)
    constexpr int LDT = B + 4;        // padded LDS row stride in floats (keeps 16-byte alignment)
    constexpr int WMAX = (B * 3 + 31) / 32;   // upper bound of position words per block row
    __shared__ __attribute__((aligned(16))) float tkept[B * LDT];
    __shared__ double rowsum[B];
    __shared__ uint32_t pos_lds[PACK ? B * WMAX : 1];
    __shared__ int viol_lds;
    const int bi = local / Kb, bj = local - bi * Kb;
    const size_t blk = (size_t)bi * Kb + bj;
    const int r = threadIdx.x / Q, q = threadIdx.x % Q;
    const int s = bi * B + r;
    const int c0 = q * LANE_COLS;                // first column of this lane inside the block
    const int k0 = bj * B + c0;
    if constexpr (PACK) {
        for (int e = threadIdx.x; e < B * WMAX; e += NTHR) pos_lds[e] = 0u;
        if (threadIdx.x == 0) {
            viol_lds = 0;
            if (bi == 0 && bj == 0) { sa.flags[0] = 1; sa.flags[1] = 0; sa.flags[2] = 0; sa.flags[3] = 0; }
        }
        __syncthreads();
    }
    float* kept_dst = &tkept[r * LDT + c0];
    uint32_t* pos_row = pos_lds + (PACK ? r * WMAX : 0);
    uint32_t bits;
    const bool vec = K % B == 0;                 // row segments are 16-byte aligned and lie wholly inside the matrix
    if (sa.m == 4) {
        bits = vec ? score_lane<B, 4, KIND, true, PACK>(sa, stg, blk, r, s, c0, k0, kept_dst, pos_row, WMAX, &viol_lds)
                   : score_lane<B, 4, KIND, false, PACK>(sa, stg, blk, r, s, c0, k0, kept_dst, pos_row, WMAX, &viol_lds);
    } else {
        bits = vec ? score_lane<B, 8, KIND, true, PACK>(sa, stg, blk, r, s, c0, k0, kept_dst, pos_row, WMAX, &viol_lds)
                   : score_lane<B, 8, KIND, false, PACK>(sa, stg, blk, r, s, c0, k0, kept_dst, pos_row, WMAX, &viol_lds);
    }
    // mask: the Q lanes of a row hold 16 bits each; pairs of lanes form one 32-bit word
    if (Q >= 2) {
        uint32_t word = bits << ((q & 1) * 16);
        word |= __shfl_xor(word, 1, 64);
        const int widx = (bj * B + c0) >> 5;
        if ((q & 1) == 0 && s < S && widx < mwpr) nm_mask[(size_t)s * mwpr + widx] = word;
    } else if (s < S) {
        // B == 16: two blocks share a mask word; each writes its own half
        uint16_t* half = reinterpret_cast<uint16_t*>(nm_mask) + ((size_t)s * mwpr) * 2;
        const int h = (bj * B) >> 4;
        half[h] = (uint16_t)bits;
        // an odd number of block columns leaves the upper half of the last word to nobody
        if (bj == Kb - 1 && (h & 1) == 0) half[h + 1] = 0;
    }
    __syncthreads();
    if (threadIdx.x < B) {
        const int row = threadIdx.x;
        double acc = 0.0;
#pragma unroll
        for (int i = 0; i < B / 4; ++i) {
            const f32x4 v = *reinterpret_cast<const f32x4*>(&tkept[row * LDT + 4 * i]);
            acc = __dadd_rn(acc, (double)v[0]);
            acc = __dadd_rn(acc, (double)v[1]);
            acc = __dadd_rn(acc, (double)v[2]);
            acc = __dadd_rn(acc, (double)v[3]);
        }
        rowsum[row] = acc;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double total = 0.0;
#pragma unroll
        for (int i0 = 0; i0 < B; i0 += 16) {     // sixteen at a time: requested together, in few registers
            double part[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) part[i] = rowsum[i0 + i];
#pragma unroll
            for (int i = 0; i < 16; ++i) total = __dadd_rn(total, part[i]);
        }
        sa.score[blk] = total;
        if constexpr (PACK) reinterpret_cast<int32_t*>(sa.stage)[blk] = viol_lds;
    }
    if constexpr (PACK) {
        uint32_t* dst = reinterpret_cast<uint32_t*>(sa.stage + stg.idxw_off) + blk * B * stg.wpr;
        for (int e = threadIdx.x; e < B * stg.wpr; e += NTHR) dst[e] = pos_lds[(e / stg.wpr) * WMAX + e % stg.wpr];
    }
}

// Compaction of a keep-flag array into ascending indices by one wave: ballot + popcount prefix.
__device__ __forceinline__ int wave_compact(const uint8_t* flags, int count, int32_t* out, int lane) {
    int written = 0;
    for (int base = 0; base < count; base += 64) {
        const int j = base + lane;
        const bool f = (j < count) && flags[j];
        const unsigned long long ballot = __ballot(f);
        const int pos = __popcll(ballot & ((1ull << lane) - 1ull));
        if (f) out[written + pos] = j;
        written += __popcll(ballot);
    }
    return written;
}

// Uniform block pruning: one workgroup per block-row keeps the k_row blocks that come first
// under (score descending, column ascending) and writes their columns in ascending order.
__global__ __launch_bounds__(256) void block_topk_rows_kernel(int Sb, int Kb, int k_row,
                                                              const double* __restrict__ score,
                                                              int32_t* __restrict__ row_ptr,
                                                              int32_t* __restrict__ col_idx) {
    __shared__ double sc[4096];
    __shared__ uint8_t kept[4096];
    const int bi = blockIdx.x, tid = threadIdx.x;
    for (int j = tid; j < Kb; j += 256) sc[j] = score[(size_t)bi * Kb + j];
    __syncthreads();
    for (int j = tid; j < Kb; j += 256) {
        const double mine = sc[j];
        int before = 0;
        for (int o = 0; o < Kb; ++o) before += (sc[o] > mine) || (sc[o] == mine && o < j);
        kept[j] = before < k_row;
    }
    __syncthreads();
    if (tid < 64) wave_compact(kept, Kb, col_idx + (size_t)bi * k_row, tid);
    if (tid == 0) {
        row_ptr[bi] = bi * k_row;
        if (bi == Sb - 1) row_ptr[Sb] = Sb * k_row;
    }
}

// Plain block pruning over the whole grid (the non-uniform baseline): keep the `budget` blocks
// that come first under (score descending, block-row ascending, column ascending).  One
// workgroup; rows may come out uneven or empty.
__global__ __launch_bounds__(1024) void block_topk_layer_kernel(int Sb, int Kb, int budget,
                                                                const double* __restrict__ score,
                                                                int32_t* __restrict__ row_ptr,
                                                                int32_t* __restrict__ col_idx) {
    __shared__ double sc[8192];
    __shared__ uint8_t kept[8192];
    __shared__ int rowcnt[1024];
    const int total = Sb * Kb, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (int a = tid; a < total; a += 1024) sc[a] = score[a];
    __syncthreads();
    for (int a = tid; a < total; a += 1024) {
        const double mine = sc[a];
        int before = 0;
        for (int o = 0; o < total; ++o) before += (sc[o] > mine) || (sc[o] == mine && o < a);
        kept[a] = before < budget;
    }
    __syncthreads();
    for (int bi = wave; bi < Sb; bi += 16) {
        int c = 0;
        for (int base = 0; base < Kb; base += 64) {
            const int j = base + lane;
            c += __popcll(__ballot((j < Kb) && kept[bi * Kb + j]));
        }
        if (lane == 0) rowcnt[bi] = c;
    }
    __syncthreads();
    if (tid == 0) {
        int pos = 0;
        for (int bi = 0; bi < Sb; ++bi) {
            const int c = rowcnt[bi];
            row_ptr[bi] = pos;
            rowcnt[bi] = pos;
            pos += c;
        }
        row_ptr[Sb] = pos;
    }
    __syncthreads();
    for (int bi = wave; bi < Sb; bi += 16) wave_compact(kept + bi * Kb, Kb, col_idx + rowcnt[bi], lane);
}

// One launch of the scoring kernel for a batch whose layers share (B, kind).
template <int KIND, bool PACK, int CAP>
static void launch_score_batch(int B, const SelBatch<ScoreLayer, CAP>& bt, hipStream_t st) {
    const unsigned grid = (unsigned)bt.first[bt.n];
    if (grid == 0) return;
    if (B == 64) score_select_kernel<64, KIND, PACK, CAP><<<grid, score_threads(64), 0, st>>>(bt);
    else if (B == 32) score_select_kernel<32, KIND, PACK, CAP><<<grid, score_threads(32), 0, st>>>(bt);
    else score_select_kernel<16, KIND, PACK, CAP><<<grid, score_threads(16), 0, st>>>(bt);
}

template <bool PACK, int CAP>
static void launch_score_kind(int sal_kind, int B, const SelBatch<ScoreLayer, CAP>& bt, hipStream_t st) {
    if (sal_kind == CRISP_SAL_GIVEN) launch_score_batch<CRISP_SAL_GIVEN, PACK>(B, bt, st);
    else if (sal_kind == CRISP_SAL_GRAD) launch_score_batch<CRISP_SAL_GRAD, PACK>(B, bt, st);
    else launch_score_batch<CRISP_SAL_MAG, PACK>(B, bt, st);
}

hipError_t launch_select(const Geometry& g, int sal_kind, int select_mode, const uint16_t* W, const float* TG,
                         uint32_t* nm_mask, int32_t* row_ptr, int32_t* col_idx, double* score, hipStream_t st) {
    SelBatch<ScoreLayer, 1> bt = {};
    bt.n = 1;
    bt.L[0] = ScoreLayer{W, TG, nm_mask, score, nullptr, nullptr, g.S, g.K, g.n, g.m};
    bt.first[1] = g.Sb * g.Kb;
    launch_score_kind<false>(sal_kind, g.B, bt, st);
    if (select_mode == CRISP_ROW_UNIFORM)
        block_topk_rows_kernel<<<g.Sb, 256, 0, st>>>(g.Sb, g.Kb, g.k_row, score, row_ptr, col_idx);
    else
        block_topk_layer_kernel<<<1, 1024, 0, st>>>(g.Sb, g.Kb, g.Sb * g.k_row, score, row_ptr, col_idx);
    return hipGetLastError();
}

// Second half of the fused select + pack (uniform rows): the workgroup of kept block (bi, t)
// works out the block choice of block-row bi on its own (k_row blocks first under score
// descending, column ascending; the Kb scores are few, so doing this once per kept block costs
// less than a launch), takes the t-th kept column in ascending order and copies that block's
// packed form from the staging area to its final place.  Results are identical to
// crisp_select_mask followed by crisp_pack.
constexpr int GATHER_THREADS = 256;
template <int CAP>
__global__ __launch_bounds__(GATHER_THREADS) void topk_gather_kernel(SelBatch<GatherLayer, CAP> bt, int B) {
    __shared__ double sc[512];
    __shared__ uint8_t kept[512];
    __shared__ int sel;
    const int li = __builtin_amdgcn_readfirstlane(layer_of<GATHER_THREADS>(bt, (int)blockIdx.x));
    const GatherLayer& L = bt.L[li];
    const int local = (int)blockIdx.x - bt.first[li];
    const int Kb = (int)(L.Kb_k_nm & 0xFFFu), k_row = (int)(L.Kb_k_nm >> 12 & 0xFFFu), Sb = L.Sb;
    const int n = (int)(L.Kb_k_nm >> 24 & 0xFu), m = (int)(L.Kb_k_nm >> 28);
    const SelStage stg = sel_stage(B, n, m, (size_t)Sb * Kb);
    const int bi = local / k_row, t = local - bi * k_row, tid = threadIdx.x;
    const int vbytes = B * stg.slots * 2, ibytes = B * stg.wpr * 4;
    for (int j = tid; j < Kb; j += GATHER_THREADS) sc[j] = L.score[(size_t)bi * Kb + j];
    __syncthreads();
    for (int j = tid; j < Kb; j += GATHER_THREADS) {
        const double mine = sc[j];
        int before = 0;
        for (int o = 0; o < Kb; ++o) before += (sc[o] > mine) || (sc[o] == mine && o < j);
        kept[j] = before < k_row;
    }
    __syncthreads();
    for (int j = tid; j < Kb; j += GATHER_THREADS) {
        if (kept[j]) {
            int pos = 0;
            for (int o = 0; o < j; ++o) pos += kept[o];
            if (pos == t) sel = j;
        }
    }
    __syncthreads();
    const int bj = sel;
    const size_t src = (size_t)bi * Kb + bj, dst = (size_t)bi * k_row + t;
    const u32x4* sv = reinterpret_cast<const u32x4*>(L.stage + stg.vals_off + src * vbytes);
    u32x4* dv = reinterpret_cast<u32x4*>(reinterpret_cast<unsigned char*>(L.vals) + dst * vbytes);
    for (int e = tid; e < vbytes / 16; e += GATHER_THREADS) dv[e] = sv[e];
    const u32x4* si = reinterpret_cast<const u32x4*>(L.stage + stg.idxw_off + src * ibytes);
    u32x4* di = reinterpret_cast<u32x4*>(reinterpret_cast<unsigned char*>(L.idxw) + dst * ibytes);
    for (int e = tid; e < ibytes / 16; e += GATHER_THREADS) di[e] = si[e];
    if (tid == 0) {
        L.col_idx[dst] = bj;
        if (t == 0) {
            L.row_ptr[bi] = bi * k_row;
            if (bi == Sb - 1) L.row_ptr[Sb] = Sb * k_row;
        }
    }
    // (n <= 2 can never put three kept elements into an aligned group of four.)  The first workgroup of a block-row looks at
    // all of its kept blocks: one access to the flag per wave that finds one, not one per block (1856 x 640 3:4, 32x32 blocks,
    // 754 kept: 11.8 us, 20 with one per block).
    if (n > 2 && t == 0) {
        bool found = false;
        for (int j = tid; j < Kb; j += GATHER_THREADS) found = found || (kept[j] && reinterpret_cast<const int32_t*>(L.stage)[(size_t)bi * Kb + j]);
        if (__ballot(found) && (tid & 63) == 0 && L.flags[0] != 0) atomicAnd(L.flags, 0);
    }
}

bool select_pack_fusable(const Geometry& g, int select_mode) {
    return select_mode == CRISP_ROW_UNIFORM && g.Kb <= 512 && g.nk > 0;
}

size_t select_pack_stage_bytes(const Geometry& g) {
    const size_t blocks = (size_t)g.Sb * g.Kb;
    return sel_stage(g.B, g.n, g.m, blocks).idxw_off + blocks * g.B * g.wpr * 4;
}

template <int CAP>
static hipError_t launch_select_pack(int n, const Geometry* g, int sal_kind, const SelPackPtrs* pp, hipStream_t st) {
    SelBatch<ScoreLayer, CAP> sb;
    SelBatch<GatherLayer, CAP> gb;
    sb.n = gb.n = n;
    sb.first[0] = gb.first[0] = 0;
    for (int i = 0; i < n; ++i) {
        unsigned char* stage = static_cast<unsigned char*>(pp[i].stage);
        sb.L[i] = ScoreLayer{pp[i].W, pp[i].TG, pp[i].nm_mask, pp[i].score, stage, pp[i].flags, g[i].S, g[i].K, g[i].n, g[i].m};
        gb.L[i] = GatherLayer{pp[i].score, stage, pp[i].vals, pp[i].idxw, pp[i].col_idx, pp[i].row_ptr, pp[i].flags, g[i].Sb,
                              (uint32_t)g[i].Kb | (uint32_t)g[i].k_row << 12 | (uint32_t)g[i].n << 24 | (uint32_t)g[i].m << 28};
        sb.first[i + 1] = sb.first[i] + g[i].Sb * g[i].Kb;
        gb.first[i + 1] = gb.first[i] + g[i].nk;
    }
    launch_score_kind<true>(sal_kind, g[0].B, sb, st);
    if (gb.first[n] > 0) topk_gather_kernel<CAP><<<(unsigned)gb.first[n], GATHER_THREADS, 0, st>>>(gb, g[0].B);
    return hipGetLastError();
}

// Fused selection + packing of up to CRISP_SELECT_BATCH layers that share (B, saliency kind) in two launches.
// stage: select_pack_stage_bytes(g[i]) bytes, 16-byte aligned.
hipError_t launch_select_pack_batch(int n, const Geometry* g, int sal_kind, const SelPackPtrs* pp, hipStream_t st) {
    return n == 1 ? launch_select_pack<1>(n, g, sal_kind, pp, st) : launch_select_pack<CRISP_SELECT_BATCH>(n, g, sal_kind, pp, st);
}

}  // namespace crisp
