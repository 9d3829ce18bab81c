// Which layer of a batched selection launch a workgroup belongs to.  Integer arithmetic only, so that it also runs in a
// host test, with a ballot over as many lanes as the workgroup has.
#pragma once

namespace crisp {

// Threads of a scoring workgroup: a block of B rows, B / 16 lanes per row.
constexpr int score_threads(int B) { return B * (B / 16); }

// first[0 .. n]: first workgroup of each layer.  The layer of workgroup `id` is the number of layers behind the first that
// begin at or before it, counted by ballots of a wave whose lanes stand for one layer each.  A workgroup of THREADS threads
// has that many lanes in its only wave where they are fewer than 64 (16 x 16 blocks: 16), so they take the layers in steps.
// ballot(p): bit l set where p(l) holds, for the lanes l of the wave.
template <int THREADS, int CAP, class BALLOT>
__host__ __device__ __forceinline__ int layer_by_ballots(int n, const int (&first)[CAP + 1], int id, BALLOT ballot) {
    static_assert(THREADS < 64 || THREADS % 64 == 0, "a wave is full, or the only one");
    constexpr int LANES = THREADS < 64 ? THREADS : 64;
    int layer = 0;
#pragma unroll
    for (int l0 = 0; l0 < CAP; l0 += LANES)
        layer += __builtin_popcountll(ballot([&](int lane) { const int l = l0 + lane; return l > 0 && l < n && id >= first[l]; }));
    return layer;
}

}  // namespace crisp
