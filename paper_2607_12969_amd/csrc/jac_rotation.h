// Rotation of the one-sided Jacobi SVD (factor.hip), in a file of its own so that
// a host program can check it.
#pragma once

namespace lrc {

// Rotation of columns p, q with al = |p|^2, be = |q|^2, ga = p . q: the
// smaller root t = tan of t^2 + 2 zeta t - 1 = 0, zeta = (be - al) / (2 ga),
// as t = sign(d) g / (|d| + sqrt(d^2 + g^2)) with d = be - al, g = 2 ga scaled
// by a power of two so that the squares stay in range.  t only has to make
// the columns orthogonal to well below the threshold (one Newton step on
// the hardware's 2^-24 estimates, 2^-46); c = 1 / sqrt(1 + t^2) and s = c t
// are to full precision (two steps), which keeps the rotation orthogonal.
// Returns false and the identity where |ga| <= tol |p| |q|.  flip: sign of
// t when d = 0.  With al and be exchanged (and flip) every step gives the same
// value or its negative, so that two lanes that hold one column each agree;
// the larger norm first in the cosine is part of that (and keeps it in range).
__device__ __forceinline__ bool jac_rotation(double al, double be, double ga, double tol, bool flip, double& t,
                                             double& c, double& s) {
    const double hi = __builtin_fmax(al, be), lo = __builtin_fmin(al, be);
    const double cosine = __builtin_fabs(ga) * __builtin_amdgcn_rsq(hi) * __builtin_amdgcn_rsq(lo);
    const bool rot = ga != 0.0 && cosine > tol;
    const int e = -__builtin_amdgcn_frexp_exp(hi);
    const double d = __builtin_amdgcn_ldexp(be - al, e), g = __builtin_amdgcn_ldexp(ga, e + 1);
    const double h2 = d * d + g * g;
    double y = __builtin_amdgcn_rsq(h2);
    y = __builtin_fma(0.5 * y, __builtin_fma(-h2 * y, y, 1.0), y);
    const double w = __builtin_fabs(d) + h2 * y;
    double z = __builtin_amdgcn_rcp(w);
    z = __builtin_fma(z, __builtin_fma(-w, z, 1.0), z);
    t = (d < 0.0 || (d == 0.0 && flip)) ? -(g * z) : g * z;
    t = rot ? t : 0.0;
    const double u = __builtin_fma(t, t, 1.0);
    c = __builtin_amdgcn_rsq(u);
    c = __builtin_fma(0.5 * c, __builtin_fma(-u * c, c, 1.0), c);
    c = __builtin_fma(0.5 * c, __builtin_fma(-u * c, c, 1.0), c);
    c = rot ? c : 1.0;
    s = c * t;
    return rot;
}

}  // namespace lrc
