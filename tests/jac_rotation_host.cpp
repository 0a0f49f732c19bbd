// Host check of the Jacobi rotation (no GPU), built and run by
// test_jac_rotation_host.py: the two lanes of a pair form it with the norms
// exchanged and must agree, also where the cosine lies on the threshold.
#include <cmath>
#include <cstdio>
#include <random>

#define __device__
#define __forceinline__ inline
static double host_rsq(double x) { return 1.0 / std::sqrt(x); }
static double host_rcp(double x) { return 1.0 / x; }
static int host_exp(double x) {
    int e = 0;
    (void)std::frexp(x, &e);
    return e;
}
#define __builtin_amdgcn_rsq host_rsq
#define __builtin_amdgcn_rcp host_rcp
#define __builtin_amdgcn_frexp_exp host_exp
#define __builtin_amdgcn_ldexp std::ldexp
#include "../paper_2607_12969_amd/csrc/jac_rotation.h"

int main() {
    std::mt19937_64 rng(3);
    std::uniform_real_distribution<double> u(0.0, 1.0);
    int bad = 0, rotated = 0, kept = 0;
    for (int i = 0; i < 200000; ++i) {
        const double al = std::exp2(40.0 * (u(rng) - 0.5)), be = i & 1 ? al * (1.0 + u(rng)) : std::exp2(40.0 * (u(rng) - 0.5));
        const double tol = (8 + i % 89) * 0x1p-53;
        double ga = tol / (host_rsq(al) * host_rsq(be));
        for (int q = 0; q < 6; ++q) ga = std::nextafter(ga, 0.0);
        for (int q = 0; q < 12; ++q, ga = std::nextafter(ga, 1e300)) {
            double t0, c0, s0, t1, c1, s1;
            const bool p = lrc::jac_rotation(al, be, ga, tol, false, t0, c0, s0);
            const bool o = lrc::jac_rotation(be, al, ga, tol, true, t1, c1, s1);
            (p ? rotated : kept) += 1;
            bad += p != o || t0 != -t1 || c0 != c1 || s0 != -s1;
        }
    }
    std::printf("%d rotated, %d kept, %d disagree\n", rotated, kept, bad);
    return bad ? 1 : (rotated > 1000 && kept > 1000 ? 0 : 2);
}
