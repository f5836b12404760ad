// hts_term.hpp -- the factors of a pair's term in double precision (also compiled
// for the host by the tests, with divisions for the hardware's approximations).
#pragma once

#include <hip/hip_runtime.h>

namespace hts {

// 1 / x from the hardware's, which has a relative error e of 2^-24: (1 - e) (1 + e + e^2)
// leaves e^3.
__device__ __forceinline__ double reciprocal(double x) {
    const double r = __builtin_amdgcn_rcp(x), e = fma(-x, r, 1.0);
    return fma(fma(e, e, e), r, r);
}

// ln(1 + u + rest) for u >= 0 and rest below u's last bit (not a number when u is not
// finite, as c then is): 1 + u = 2^e m, m in [0.85, 1.7), f = f0 + c with f0 = m - 1 and c what the
// rounding of 1 + u and rest left out, and with s = f / (2 + f) ln(1 + f) =
// 2 artanh s = f - s (f - 2 s^2 g(s^2)), g(z) = 1/3 + z/5 + z^2/7 + ... by its Chebyshev
// interpolant of degree 7 on [0, (0.7 / 2.7)^2] (relative error of the result
// 6e-17).  f0 is exact and joins the sum last: the rounding of f then counts by s only.
// About 30 instructions without a branch where the library's log1p takes 120 in
// sums of two doubles.
__device__ __forceinline__ double log1p_pos(double u, double rest = 0.0) {
    const double y = 1.0 + u;
    const int hi = __double2hiint(y);
    const int e = (hi - 0x3feb3333) >> 20;
    const double m = __hiloint2double(hi - (e << 20), __double2loint(y));
    const double f0 = m - 1.0;
    const double c = __builtin_amdgcn_ldexp(u - (y - 1.0) + rest, -e);
    const double f = f0 + c;
    const double s = f * reciprocal(2.0 + f), z = s * s;
    double g = 0.07527378486732582;
    g = fma(g, z, 0.06478276194288947);
    g = fma(g, z, 0.07703270293461335);
    g = fma(g, z, 0.09090559165270742);
    g = fma(g, z, 0.1111111714554286);
    g = fma(g, z, 0.14285714234773572);
    g = fma(g, z, 0.20000000000163445);
    g = fma(g, z, 0.3333333333333325);
    const double l = f0 + fma(-s, fma(-2.0, z * g, f), c);
    const double de = (double)e;
    return fma(de, 0.6931471805599453, fma(de, 2.3190468138462996e-17, l));
}

// The factors of a pair's term in double: d = acosh(1 + t) = ln(1 + t + sqrt(t (t +
// 2))), which has full relative accuracy for small t (the argument of eq. (8) is
// carried as t = gamma - 1, never gamma), w and d / sinh d.  One
// reciprocal square root gives sinh d and its reciprocal (Goldschmidt's steps);
// 1e-300 keeps it finite at t = 0 and is below the last bit of any other x.
// With the library's log1p, square root and divisions the exact gradient of n =
// 20000 points took 1.43 ms, now 0.63.
// rms error in units of 2^-53, with a correctly rounded logarithm, root and divisions and
// so: t in [0.01, 1] w 0.732 and 0.699, d / sinh d 0.668 and 0.629; [1, 100] 1.042 and
// 0.994, 0.752 and 0.739; elsewhere the same or less.  (Without what the sum of t and
// sinh d leaves out, and with f for f0 + c in the last sum, d / sinh d had 0.702 in the
// first of these.)
__device__ __forceinline__ double pair_weight(double t, double &w, double &ratio) {
    const double x = fma(t, t + 2.0, 1e-300);
    const double rs = __builtin_amdgcn_rsq(x);
    double sh = x * rs, h = 0.5 * rs;
    const double c = fma(-h, sh, 0.5);
    sh = fma(sh, c, sh);
    h = fma(h, c, h);
    sh = fma(fma(-sh, sh, x), h, sh);
    const double u = sh + t;  // (sinh d is the larger)
    const double d = log1p_pos(u, t - (u - sh));
    w = reciprocal(fma(d, d, 1.0));
    const double r = d * (h + h);
    ratio = fma(fma(-sh, r, d), h + h, r);
    return d;
}

}  // namespace hts
