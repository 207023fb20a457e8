// Fully polarised LSDA of one FLO density, E_xc[rho_i, 0] of Eq. 1 (Sec. III):
// Slater exchange and the PW92 correlation interpolation at zeta = 1.
//   exchange: eps_x = -(3/4)(6/pi)^(1/3) rho^(1/3), v_x = (4/3) eps_x
//   correlation: G(rs) = -2A (1 + alpha1 rs) ln(1 + 1 / q1(rs)),
//     q1 = 2A (beta1 rs^(1/2) + beta2 rs + beta3 rs^(3/2) + beta4 rs^2),
//     A = 0.015545, alpha1 = 0.20548, beta1..4 = 14.1189, 6.1977, 3.3662, 0.62517;
//     v_c = eps_c - (rs/3) d eps_c / d rs (no zeta term at zeta = 1).
// The passes that evaluate it once per node and orbital are bound by its
// FP64 operations, so it has one sixth root (every power of rho is a product
// of it), one reciprocal (three denominators share it) and one logarithm by a
// short polynomial, and no branch: about 65 operations a density, where
// separate cube and square roots, reciprocals and the library's log1p took
// about 150.
#pragma once

#include "kernels.h"

namespace fsic {

// (6/pi)^(1/3) and (3/(4 pi))^(1/3) and its square root
constexpr double kSixOverPiCbrt = 1.2407009817988000333;
constexpr double kRsCoef = 0.62035049089940001667;
constexpr double kRsCoefSqrt = 0.78762331789974325;

// x^(-1/6), x > 0 in single-precision range: Newton's method for y^-6 = x,
// y <- y + y (1 - x y^6) / 6, two steps from a single-precision value
__device__ __forceinline__ double newton_inv_root6(double x) {
    double y = (double)__builtin_amdgcn_exp2f(-(1.0f / 6.0f) * __builtin_amdgcn_logf((float)x));
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const double y2 = y * y;
        y = fma(y * (1.0 / 6.0), fma(-x * y2, y2 * y2, 1.0), y);
    }
    return y;
}

// 1/x: Newton's method for 1/y = x, y <- y + y (1 - x y), two steps from the
// hardware's estimate
__device__ __forceinline__ double newton_recip(double x) {
    double y = __builtin_amdgcn_rcp(x);
#pragma unroll
    for (int k = 0; k < 2; ++k) y = fma(y, fma(-x, y, 1.0), y);
    return y;
}

// energies per particle and potentials at one density; rho <= floor: all zero
__device__ __forceinline__ void lsda_pol(double rho, double floor, double &ex, double &ec, double &vx,
                                         double &vc) {
    constexpr double A = 0.015545, a1 = 0.20548;
    constexpr double b1 = 14.1189, b2 = 6.1977, b3 = 3.3662, b4 = 0.62517;
    const bool on = rho > floor;
    const double d = on ? rho : 1.0;
    const double t = newton_inv_root6(d);  // rho^(-1/6)
    const double y = t * t;                // rho^(-1/3)
    const double y2 = y * y, ra = d * y2;
    const double r13 = fma(y2 * (1.0 / 3.0), fma(-ra * ra, ra, d), ra);  // rho^(1/3), one more step
    const double rs = kRsCoef * y, s = kRsCoefSqrt * t;
    const double is = (1.0 / kRsCoefSqrt) * (r13 * t);  // rs^(-1/2) ~ rho^(1/6)
    const double q1 = s * fma(s, fma(s, fma(s, 2.0 * A * b4, 2.0 * A * b3), 2.0 * A * b2), 2.0 * A * b1);
    const double q1p = fma(A * b1, is, fma(s, fma(s, 4.0 * A * b4, 3.0 * A * b3), 2.0 * A * b2));  // d q1 / d rs
    // ln(1 + 1/q1) = e ln 2 + 2 artanh(g), g = (w - Q) / (w + Q), w = q1 + 1,
    // Q = 2^e q1, with e such that w / Q is within a factor sqrt 2 of 1 (e = 0
    // for low densities, where w - Q is 1 exactly); artanh(g) = g + g^3 p(g^2),
    // p interpolating the series on [0, (sqrt 2 - 1)^2 / (sqrt 2 + 1)^2]
    // (relative error 5e-18).  1 / (q1 (q1 + 1)) = (1/q1)^2 / (1 + 1/q1) shares
    // the reciprocal.
    const float ef = __builtin_rintf(__builtin_amdgcn_logf(1.0f + __builtin_amdgcn_rcpf((float)q1)));
    const int e = (int)ef;
    const double w = q1 + 1.0, Q = __builtin_amdgcn_ldexp(q1, e);
    const double d1 = q1 * w, d2 = w + Q;
    const double inv = newton_recip(d1 * d2);
    const double i1 = inv * d2;
    const double g = (e == 0 ? 1.0 : w - Q) * (inv * d1);
    const double z = g * g;
    double p = 0.073082927124443114;
    p = fma(p, z, 0.076658553091053863);
    p = fma(p, z, 0.090914447278374735);
    p = fma(p, z, 0.11111105565129939);
    p = fma(p, z, 0.14285714313001635);
    p = fma(p, z, 0.19999999999949722);
    p = fma(p, z, 0.33333333333333348);
    const double g2 = g + g;
    const double lg = fma((double)ef, 0.69314718055994531, fma(g2 * z, p, g2));
    const double q0 = fma(-2.0 * A * a1, rs, -2.0 * A);
    const double c = q0 * lg;
    // d eps_c / d rs = -2A alpha1 lg - q0 q1p / (q1 (q1 + 1))
    const double dec = fma(-(q0 * q1p), i1, (-2.0 * A * a1) * lg);
    ex = on ? -0.75 * kSixOverPiCbrt * r13 : 0.0;
    vx = on ? -kSixOverPiCbrt * r13 : 0.0;
    ec = on ? c : 0.0;
    vc = on ? fma(rs * dec, -1.0 / 3.0, c) : 0.0;
}

// v_x + v_c at one density
__device__ __forceinline__ double vxc_pol(double rho, double floor) {
    double ex, ec, vx, vc;
    lsda_pol(rho, floor, ex, ec, vx, vc);
    return vx + vc;
}

}  // namespace fsic
