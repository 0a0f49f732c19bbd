// Host sweeps over apply plans (no GPU), built and run by
// test_apply_plan_host.py; each prints the plans that fail it.
//   scratch  every FP32 call whose scratch_bytes the allocation-free entry takes
//            fits its scratch in the plan that runs
//   memory   where only the memory of the plan without the split is free, the
//            split's reservation still succeeds within it
//   route    the FP32 split runs where it was measured to gain, not where it lost
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <random>

#include "../include/lrc.h"
#include "../paper_2607_12969_amd/csrc/lrc_internal.h"

using namespace lrc;

namespace {
const size_t kLimit = (size_t)LRC_NOALLOC_SCRATCH_BYTES;
int bad = 0;
long split = 0, cut = 0;

void failed(int64_t m, int64_t n, int64_t k, int64_t b, size_t need, size_t limit) {
    ++bad;
    std::printf("%lld x %lld k %lld b %lld: %zu of %zu\n", (long long)m, (long long)n, (long long)k, (long long)b, need,
                limit);
}

void memory(int64_t m, int64_t n, int64_t k, int64_t b) {
    if (k > std::min(m, n)) return;
    const void* p = reinterpret_cast<const void*>((uintptr_t)0x10000);
    const ApplyPlan whole = plan_apply(m, n, k, b, P32, 0, p, p, p);
    const auto general = [&] { return plan_apply(m, n, k, b, P32, 0, p, p, p, false); };
    const size_t full = apply_workspace_bytes(whole), least = apply_workspace_bytes(general());
    split += whole.x3;
    for (size_t room : {full, (full + least) / 2, least}) {
        ApplyPlan plan = whole;
        size_t got = 0;
        int calls = 0;
        const hipError_t e = reserve_apply(
            plan, m, b,
            [&](size_t bytes) {
                ++calls;
                got = bytes;
                return bytes <= room ? hipSuccess : hipErrorOutOfMemory;
            },
            general);
        if (e != hipSuccess || got != apply_workspace_bytes(plan) || (room >= full && calls != 1))
            failed(m, n, k, b, got, room);
        cut += calls > 1;
    }
}

void scratch(int64_t m, int64_t n, int64_t k, int64_t b) {
    if (k > std::min(m, n)) return;
    const void* p = reinterpret_cast<const void*>((uintptr_t)0x10000);
    ApplyPlan plan = plan_apply(m, n, k, b, P32, 0, p, p, p);
    if (plan.scratch_bytes > kLimit) return;
    if (plan.x3) {
        ++split;
        cut += apply_workspace_bytes(plan) > kLimit;
        x3_panels(plan, m, b, kLimit);
    }
    const size_t need = apply_workspace_bytes(plan);
    if (need > kLimit || (plan.x3 && (plan.bpanel < 1 || plan.mpanel < 1 || plan.vgroup < 1)))
        failed(m, n, k, b, need, kLimit);
}
}  // namespace

struct Route {
    int64_t m, n, k, b;
    bool split;
};
// times of the split over those of the FP32 instruction's plan beside each size
const Route kRoutes[] = {
    {8192, 8192, 257, 4096, true},    // 0.60
    {2003, 1733, 41, 2047, true},     // 0.86
    {65536, 4096, 513, 4096, true},   // 0.72
    {4000, 30000, 16, 4095, true},    // 0.45
    {2500, 2500, 24, 8192, true},     // 0.93
    {8192, 8192, 129, 1024, true},    // 0.84
    {11121, 25030, 16, 5440, false},  // 1.22
    {30000, 4000, 8, 2048, false},    // 1.18
    {4000, 30000, 24, 1024, false},   // 1.13
    {2000, 16000, 41, 1024, false},   // 1.10
    {16000, 1000, 41, 513, false},    // 1.19
    {1200, 6000, 97, 1024, false},    // 1.16
    {1200, 6000, 64, 1023, false},    // 1.10
    {16384, 16384, 1, 4096, false},   // sums of three products and less: larger errors
    {16384, 16384, 3, 4095, false},
    {16384, 16384, 2, 8191, false},
};

void route(const Route& c) {
    // factors of a rank that is no multiple of four and odd batches are misaligned by themselves
    const void* p = reinterpret_cast<const void*>((uintptr_t)0x10000);
    const ApplyPlan plan = plan_apply(c.m, c.n, c.k, c.b, P32, 0, p, p, p);
    if ((plan.x3 != 0) != c.split) failed(c.m, c.n, c.k, c.b, plan.x3, c.split);
}

int main(int argc, char** argv) {
    if (argc != 2) return 3;
    if (std::strcmp(argv[1], "route") == 0) {
        for (const Route& c : kRoutes) route(c);
        return bad ? 1 : 0;
    }
    const auto check = std::strcmp(argv[1], "scratch") == 0 ? scratch : memory;
    // one split of the planes of V just above a quarter of the scratch
    check(8194, 47657, 332, 5388);
    check(8029, 47634, 336, 5560);
    check(292436, 103217, 352, 7104);
    check(47631, 47631, 336, 8192);
    std::mt19937_64 rng(1);
    auto size = [&](double lo, double hi) {
        return (int64_t)std::exp(std::uniform_real_distribution<double>(std::log(lo), std::log(hi))(rng));
    };
    for (int i = 0; i < 400000; ++i) check(size(128, 400000), size(16, 400000), size(1, 5000), size(512, 60000));
    // splits at the largest bytes of V's planes: n a multiple of what fills them
    for (int64_t k = 17; k <= 4400; k += 5)
        for (int64_t q = 1; q <= 12; ++q) {
            const int64_t kpad = round_up(k, 16) + 16, n = q * ((int64_t)(16 << 20) / (6 * kpad));
            for (int64_t b : {512, 1024, 4096, 8192})
                for (int64_t m : {4400, 65536}) check(m, n + (k & 31), k, b);
        }
    std::printf("%ld split plans, %ld cut, %d do not fit\n", split, cut, bad);
    return bad ? 1 : (split > 1000 && cut > 100 ? 0 : 2);
}
