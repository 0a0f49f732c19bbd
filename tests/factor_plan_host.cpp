// Host check of the factorization products' routes (no GPU), built and run by
// test_apply_plan_host.py: A^T Q straight from memory only where that was
// measured to be faster, and without a workspace there; the sketch's tiles.
#include <cstdio>

#include "../paper_2607_12969_amd/csrc/lrc_internal.h"

using namespace lrc;

int main() {
    struct Case {
        int64_t nq, cols, K;
        bool slim;
    };
    // times of the kernel over those of the split tiles beside each size
    const Case cases[] = {
        {74, 114688, 512, true},   // 0.77
        {74, 65536, 8192, true},   // 0.71
        {74, 49152, 256, true},    // 0.87
        {74, 32768, 8192, false},  // 1.39
        {74, 40002, 8192, false},  // 1.14
        {74, 81920, 8192, false},  // 1.08
        {60, 32768, 8192, false},  // 2.14
        {60, 114688, 2048, false}, // 1.22
        {40, 32768, 2048, false},  // 1.72
        {40, 114688, 8192, false}, // 1.15
        {20, 114688, 512, true},   // 0.85
        {12, 65536, 256, true},    // 0.74
        {20, 32768, 2048, false},  // 1.54
        {20, 49152, 8192, false},  // 1.33
        {12, 65536, 8192, false},  // 1.07
        {20, 400000, 2048, false}, // 1.07
        {90, 32768, 8192, false},  // 2.05
        {96, 81920, 2048, false},  // 1.39
        {74, 32766, 8192, false}, {74, 1000, 512, false}, {20, 8192, 8192, false},
    };
    int bad = 0;
    for (const Case& c : cases) {
        const bool slim = gemm_tn_workspace_bytes(c.nq, c.cols, c.K) == 0 && tn_slim_takes(c.nq, c.cols, c.K);
        const bool tiles = !tn_slim_takes(c.nq, c.cols, c.K);
        if (c.slim ? !slim : !tiles) {
            ++bad;
            std::printf("%lld of %lld columns, K %lld\n", (long long)c.nq, (long long)c.cols, (long long)c.K);
        }
    }
    // A Omega^T for 81 to 96 test vectors: 1536 workgroups of 96-row tiles (six
    // fragments a wave leave one workgroup per compute unit, 1.05 to 1.19 times
    // their time), 512 of slim tiles below
    const int64_t rows = 8192, K = 32768, tiles = rows / 64;
    for (int64_t nw : {65, 80, 81, 96}) {
        const int64_t bm = nw > 80 ? 96 : 80, splits = (nw > 80 ? 1536 : 512) / tiles;
        if (gemm_nt_workspace_bytes(nw, rows, K) != (size_t)(tiles * splits * bm * 64 * 8)) {
            ++bad;
            std::printf("sketch of %lld\n", (long long)nw);
        }
    }
    return bad ? 1 : 0;
}
