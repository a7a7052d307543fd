// FP64 kernel differences of the fills without divisions or square roots.
#pragma once

#include "p2_device.h"

namespace mbem {

// closed-form kernel constants, passed by value (uniform operands)
struct PairConst {
    double ka, ki_re, ki_im, eps_re, eps_im, mu_re, mu_im, kmax;
};

// 1 / sqrt(x) for x > 0: the hardware estimate (at least 24 bits) and one
// third-order step, y (1 + e/2 + 3 e^2/8) with e = 1 - x y^2.
__device__ __forceinline__ double rsqrt64(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

// The closed forms of kernel_scalars times w, for one real exterior and one
// complex interior wavenumber (units: eps_a = mu_a = 1).  With t = k R,
// e = e^{it} / (4 pi R^3), g = e (1 - i t) and h = e t^2 per medium:
//   D0 = h_a - h_i, dg = g_a - g_i, df = 3 dg - D0,
//   G_eps = -R (g_a - eps_i g_i), G_mu = -R (g_a - mu_i g_i).
__device__ __forceinline__ KScal<double> scalars_closed64(const PairConst &K, double R, double rinv, double w) {
    const double r3 = w * 0.079577471545947667884 * rinv * (rinv * rinv);
    double sn, cs;
    const double ta = K.ka * R;
    sincos_t(ta, &sn, &cs);
    const cx<double> ea = {r3 * cs, r3 * sn};
    const cx<double> ga = {fma(ea.im, ta, ea.re), fma(-ea.re, ta, ea.im)};
    const double ta2 = ta * ta;
    const double tr = K.ki_re * R, ti = K.ki_im * R;
    sincos_t(tr, &sn, &cs);
    const double am = K.ki_im == 0.0 ? r3 : r3 * exp(-ti);
    const cx<double> ei = {am * cs, am * sn};
    const double u = 1.0 + ti;
    const cx<double> gi = {fma(ei.im, tr, ei.re * u), fma(-ei.re, tr, ei.im * u)};
    const cx<double> t2 = {fma(tr, tr, -(ti * ti)), 2.0 * tr * ti};
    KScal<double> o;
    o.D0 = {fma(ta2, ea.re, fma(t2.im, ei.im, -(t2.re * ei.re))),
            fma(ta2, ea.im, -fma(t2.re, ei.im, t2.im * ei.re))};
    o.dg = ga - gi;
    o.df = {fma(3.0, o.dg.re, -o.D0.re), fma(3.0, o.dg.im, -o.D0.im)};
    o.Ge = {-R * fma(K.eps_im, gi.im, fma(-K.eps_re, gi.re, ga.re)),
            -R * fma(-K.eps_im, gi.re, fma(-K.eps_re, gi.im, ga.im))};
    o.Gm = {-R * fma(K.mu_im, gi.im, fma(-K.mu_re, gi.re, ga.re)),
            -R * fma(-K.mu_im, gi.re, fma(-K.mu_re, gi.im, ga.im))};
    return o;
}

}  // namespace mbem
