// Twelve weighted kernel values of the Galerkin fill at a test point
// (x, n, t_a, s_a) and a trial point (y, t_b) (eqs. kappa1_alphabeta,
// kappa2_alpha_beta):
//   kappa1_ab = (D0 - dg)(s_a.t_b) + df (s_a.R)(R.t_b)
//   kappa2_ab = G_chi [(t_a.t_b)(n.R) - (t_a.R)(n.t_b)],  R = (x - y)/|x - y|
// output order c = 4 op + 2 a + b, op: K1, K2^eps, K2^mu.
#pragma once

#include "p2_device.h"

namespace mbem {

template <typename T>
__device__ __forceinline__ void kappa_combine(const KScal<T> &s, vec3<T> Rh, vec3<T> n,
                                              const vec3<T> ta[2], const vec3<T> sa[2],
                                              const vec3<T> tb[2], T ww, cx<T> out[12]) {
    const cx<T> A = s.D0 - s.dg;
    const T nR = dot(n, Rh);
    T tRy[2], ntb[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) { tRy[b] = dot(tb[b], Rh); ntb[b] = dot(n, tb[b]); }
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        const T sR = dot(sa[a], Rh), tR = dot(ta[a], Rh);
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const T st = dot(sa[a], tb[b]);
            const T g2 = dot(ta[a], tb[b]) * nR - tR * ntb[b];
            const cx<T> k1 = st * A + (sR * tRy[b]) * s.df;
            out[0 + 2 * a + b] = ww * k1;
            out[4 + 2 * a + b] = (ww * g2) * s.Ge;
            out[8 + 2 * a + b] = (ww * g2) * s.Gm;
        }
    }
}

template <typename T>
__device__ __forceinline__ void kappa12(const KernelConst &K, vec3<T> x, vec3<T> n,
                                        const vec3<T> ta[2], const vec3<T> sa[2],
                                        vec3<T> y, const vec3<T> tb[2], T ww,
                                        cx<T> out[12]) {
    vec3<T> Rv = x - y;
    const T R = sqrt(dot(Rv, Rv));
    const vec3<T> Rh = ((T)1 / R) * Rv;
    kappa_combine<T>(kernel_scalars<T>(K, R), Rh, n, ta, sa, tb, ww, out);
}

}  // namespace mbem
