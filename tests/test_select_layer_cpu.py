"""Which layer a workgroup of a batched selection launch takes, on the CPU: the header that counts it by ballots, compiled
by the host compiler and asked for every workgroup of random batches of every length, with ballots over exactly the lanes
that a workgroup of the launch has (16 x 16 blocks: sixteen)."""
import os
import subprocess

from paper_2311_14272_amd import synth

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2311_14272_amd", "csrc")

HARNESS = r"""
#define __host__
#define __device__
#define __forceinline__ inline
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include "select_layer.h"
using namespace crisp;
static long long bad, asked;
template <int THREADS, int CAP>
static void ask(const char* what, const int (&first)[CAP + 1], int n) {
    int want = 0;
    for (int id = 0; id < first[n]; ++id) {
        while (id >= first[want + 1]) ++want;
        int waves = 0;
        for (int wave = 0; wave * 64 < THREADS; ++wave, ++waves) {
            const int lanes = std::min(64, THREADS - wave * 64);
            const int got = layer_by_ballots<THREADS, CAP>(n, first, id, [&](auto p) {
                uint64_t bits = 0;
                for (int lane = 0; lane < lanes; ++lane) bits |= (uint64_t)(p(lane) ? 1 : 0) << lane;
                return bits;
            });
            if (got != want && ++bad <= 5) printf("%s: %d threads, %d layers, workgroup %d: layer %d, not %d\n", what, THREADS, n, id, got, want);
            ++asked;
        }
    }
}
template <int B, int CAP>
static void all_of(const char* what, const int (&first)[CAP + 1], int n) {
    ask<score_threads(B), CAP>(what, first, n);
    ask<256, CAP>(what, first, n);                            // the second launch of the pair
}
int main(int argc, char** argv) {
    constexpr int CAP = CAPACITY;
    static_assert(score_threads(16) == 16 && score_threads(32) == 64 && score_threads(64) == 256, "a lane takes 16 columns of a row");
    // (the entries behind the last layer are whatever the stack held)
    for (int n = 1; n <= CAP; ++n) for (int round = 0; round < 20; ++round) {
        int first[CAP + 1];
        for (int i = 0; i <= CAP; ++i) first[i] = rand() - RAND_MAX / 2;
        first[0] = 0;
        for (int i = 0; i < n; ++i) first[i + 1] = first[i] + 1 + (rand() % 3 ? rand() % 4 : rand() % 300);
        all_of<16, CAP>("random", first, n);
        all_of<32, CAP>("random", first, n);
        all_of<64, CAP>("random", first, n);
    }
    int first[CAP + 1] = {0}, n = 0;
    for (int i = 1; i < argc && n < CAP; ++i, ++n) first[n + 1] = first[n] + atoi(argv[i]);
    all_of<16, CAP>("network", first, n);
    printf("%lld bad of %lld\n", bad, asked);
    return bad != 0 || asked == 0;
}
"""


def test_every_workgroup_finds_its_layer(tmp_path):
    with open(os.path.join(CSRC, "crisp_internal.h")) as f:
        cap = next(line.split()[2] for line in f if line.startswith("#define CRISP_SELECT_BATCH"))
    src = tmp_path / "ask.cpp"
    src.write_text(HARNESS)
    exe = tmp_path / "ask"
    subprocess.run(["g++", "-O2", "-std=c++17", "-DCAPACITY=" + cap, "-I" + CSRC, str(src), "-o", str(exe)], check=True)
    blocks = [-(-L.S // 16) * -(-L.K // 16) for L in synth.resnet50(1, synth.SEED_BASE).layers]
    assert len(blocks) == 53
    r = subprocess.run([str(exe)] + [str(b) for b in blocks], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout
