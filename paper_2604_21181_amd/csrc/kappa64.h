// FP64 kernel differences of the fills: closed forms from a root and an inverse
// root, without divisions (the series below max|k| R = 1/2 divide, as before).
#pragma once

#include <algorithm>
#include <cmath>

#include "p2_device.h"

namespace mbem {

// closed-form kernel constants, passed by value (uniform operands)
struct PairConst {
    double ka, ki_re, ki_im, eps_re, eps_im, mu_re, mu_im, kmax;
    double ka2, ki2_re, ki2_im;    // their squares
};
inline PairConst pair_const(double2 ka, double2 ki, double2 eps, double2 mu) {
    return {ka.x, ki.x, ki.y, eps.x, eps.y, mu.x, mu.y, std::max(std::hypot(ka.x, ka.y), std::hypot(ki.x, ki.y)),
            ka.x * ka.x, std::fma(ki.x, ki.x, -(ki.y * ki.y)), 2.0 * ki.x * ki.y};
}

// sqrt(x) and 1 / sqrt(x) for x > 0: the hardware estimate y (at least 24 bits)
// and one third-order step, y (1 + e/2 + 3 e^2/8) with e = 1 - x y^2 formed
// from both halves of the product x y; the root is corrected by its own
// residual.  Both are within an ulp, mostly the nearest number, as a square
// root and a division are.  The residuals' four operations are needed: a
// distance taken as x times the rounded inverse root, which every scalar of a
// pair inherits, raised the error of K1 by 2 to 12 %.
struct Root64 {
    double r, inv;
};
__device__ __forceinline__ Root64 root64(double x) {
    const double y = __builtin_amdgcn_rsq(x), h = x * y;
    const double e = fma(-fma(x, y, -h), y, fma(-h, y, 1.0));
    const double inv = fma(y * e, fma(0.375, e, 0.5), y), r = x * inv;
    return {fma(0.5 * inv, fma(-r, r, x), r), inv};
}

// e^{ikR} of both media and what the scalars are made of (units: eps_a = mu_a =
// 1, k_a real).  With t = k R and e = e^{it} per medium: g = e (1 - i t),
// f = e (3 - 3 i t - t^2), d = k_a^2 e_a - k_i^2 e_i.  Each medium's polynomial
// is formed before the media are subtracted, and the common powers of 1/R come
// last: df as 3 dg - D0, or e^{it}/R^3 rounded before its polynomials, leaves
// errors of the media's terms where their difference is small.
struct Media64 {
    cx<double> ga, gi, fa, fi, d, ha, hi;   // h = e t^2
    double ta2;
    cx<double> ti2;                          // t^2
};
__device__ __forceinline__ Media64 media64(const PairConst &K, double R) {
    Media64 m;
    double sn, cs;
    const double ta = K.ka * R;
    sincos_t(ta, &sn, &cs);
    const cx<double> ea = {cs, sn};
    m.ta2 = ta * ta;
    const double tr = K.ki_re * R, ti = K.ki_im * R;
    sincos_t(tr, &sn, &cs);
    const double am = K.ki_im == 0.0 ? 1.0 : exp(-ti);
    const cx<double> ei = {am * cs, am * sn};
    m.ti2 = {fma(tr, tr, -(ti * ti)), 2.0 * tr * ti};
    m.ga = ea * cx<double>{1.0, -ta};
    m.gi = ei * cx<double>{1.0 + ti, -tr};
    m.fa = ea * cx<double>{3.0 - m.ta2, -3.0 * ta};
    m.fi = ei * cx<double>{fma(3.0, ti, 3.0) - m.ti2.re, fma(-3.0, tr, -m.ti2.im)};
    m.ha = m.ta2 * ea;
    m.hi = m.ti2 * ei;
    m.d = K.ka2 * ea - cx<double>{K.ki2_re, K.ki2_im} * ei;
    return m;
}

// The closed forms of kernel_scalars times w:
//   D0 = d / (4 pi R), df = (f_a - f_i) / (4 pi R^3), dg = (g_a - g_i) / (4 pi R^3),
//   G_eps = -(g_a - eps_i g_i) / (4 pi R^2), G_mu = -(g_a - mu_i g_i) / (4 pi R^2).
__device__ __forceinline__ KScal<double> scalars_closed64(const PairConst &K, double R, double rinv, double w) {
    const double r1 = w * 0.079577471545947667884 * rinv, r2 = r1 * rinv, r3 = r2 * rinv;
    const Media64 m = media64(K, R);
    KScal<double> o;
    o.D0 = r1 * m.d;
    o.df = r3 * (m.fa - m.fi);
    o.dg = r3 * (m.ga - m.gi);
    o.Ge = (-r2) * (m.ga - cx<double>{K.eps_re, K.eps_im} * m.gi);
    o.Gm = (-r2) * (m.ga - cx<double>{K.mu_re, K.mu_im} * m.gi);
    return o;
}

}  // namespace mbem
