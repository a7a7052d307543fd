// Shape gradient of sigma_ext by the adjoint method (extension of Sec. 6).
//
// With the solution x of Z x = b and lambda of Z^T lambda = g (g the
// far-field functional, sigma = (4 pi / k) Im g^T x), the derivative of
// sigma with respect to any geometric parameter is (4 pi / k) times that of
//     Phi = Im( g^T x + lambda^T b - lambda^T Z x )      (x, lambda frozen).
// Every term of Phi is a sum over quadrature points (right-hand side, far
// field, mass) or point pairs (dense blocks, Sec. 4) of an expression in
// the point's position, weight W = w J, normal n and frame t1, t2 (Sec. 3),
// with the current coefficients interpolated by the shape functions:
//   test point:  p_1 = L0 t1 + L1 t2,  p_2 = L2 t1 + L3 t2  (from lambda),
//                u_a = p_a x n  (= sum_alpha L s_alpha),
//   trial point: v_j = X0 t1 + X1 t2,  v_m = X2 t1 + X3 t2  (from x).
// The point-pair integrand of lambda^T Z x (eqs. kappa1/kappa2 summed over
// alpha, beta with these weights) is, with R the unit vector between the points,
//   F = (i/w) [A (u1.vj - u2.vm) + df ((u1.R)(R.vj) - (u2.R)(R.vm))]
//     + G_eps u1.(vm x R) + G_mu u2.(vj x R)
//     = u1.S1 + u2.S2 = vj.Hj + vm.Hm
// with A = D0 - dg (p.v (n.R) - (p.R)(n.v) = (p x n).(v x R)): linear in every
// vector, so the adjoints of a point's vectors, normal and weight follow from
// the sums of S (over trial points) and of H (over test points), and only the
// position's adjoint is formed pair by pair.  Reverse mode: adjoints of the point quantities are
// accumulated per quadrature point (regular rule) or per singular pair
// (Sauter-Schwab points), carried back through the P2 map and the
// Gram-Schmidt frame to node positions and nodal tangents, and through the
// nodal triads and metric-weighted normals to node positions.  The pair
// classes and the choice of reference vector are held fixed.
// Node-attached tangents (NODAL): the point vectors are p = m - (m.n) n with
// m = sum_k N_k sum_b c_kb t_b,k; their adjoints are kept as vectors and
// carried back through that projection to the normal and to the nodal
// tangents, which then go through the nodal triads as above.
#include <cmath>

#include "mbem_internal.h"
#include "kappa64.h"
#include "p2_device.h"
#include "ssq_map.h"
#include "wave.h"

namespace mbem {

using cxd = cx<double>;

// ------------------------------------------------------- complex vectors --
struct cv3 {
    cxd x, y, z;
};
__device__ inline cv3 operator+(cv3 a, cv3 b) { return {a.x + b.x, a.y + b.y, a.z + b.z}; }
__device__ inline cv3 operator-(cv3 a, cv3 b) { return {a.x - b.x, a.y - b.y, a.z - b.z}; }
__device__ inline cv3 operator*(cxd s, cv3 a) { return {s * a.x, s * a.y, s * a.z}; }
__device__ inline cv3 operator*(cxd s, dvec3 a) { return {a.x * s, a.y * s, a.z * s}; }
__device__ inline cv3 operator*(double s, cv3 a) { return {s * a.x, s * a.y, s * a.z}; }
__device__ inline cxd cdot(cv3 a, dvec3 b) { return b.x * a.x + b.y * a.y + b.z * a.z; }
__device__ inline cxd cdot(cv3 a, cv3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ inline cv3 ccross(dvec3 a, cv3 b) {
    return {a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}
__device__ inline cv3 ccross(cv3 a, dvec3 b) {
    return {b.z * a.y - b.y * a.z, b.x * a.z - b.z * a.x, b.y * a.x - b.x * a.y};
}
__device__ inline cv3 ccross(cv3 a, cv3 b) {
    return {a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}
__device__ inline dvec3 im3(cv3 a) { return {a.x.im, a.y.im, a.z.im}; }

// ------------------------------ kernel differences and their R-derivatives --
// times i/w (a, d: A = D0 - dg and df) and d/dR of each
struct KScalD {
    cxd a, ap, d, dp, Ge, Gep, Gm, Gmp;
};

__device__ inline void horner_d(const double *c, double R, cxd &S, cxd &Sp) {
    S = {c[2 * kSeriesTerms], c[2 * kSeriesTerms + 1]};
    Sp = {0.0, 0.0};
    for (int n = kSeriesTerms - 1; n >= 0; --n) {
        Sp = cxd{Sp.re * R + S.re, Sp.im * R + S.im};
        S = cxd{S.re * R + c[2 * n], S.im * R + c[2 * n + 1]};
    }
}

struct ShapeConst {
    PairConst kc;
    cxd iw;
};

// Same branches as kernel_scalars: Taylor series (Ks) below max|k| R = 1/2,
// closed forms above.  Per medium, with t = k R and e = e^{it} / (4 pi R^3),
//   g = e (1 - i t), h = e t^2, q = g t^2:  D0 = h, f = 3 g - h,
//   R g' = -f,  R f' = q - 3 f,  R D0' = -q,
// and (R g)' = h - 2 g in G_chi = -R (g_a - chi_i g_i).
__device__ __forceinline__ KScalD kernel_scalars_dr(const ShapeConst &C, const KernelConst &Ks, double R,
                                                    double rinv) {
    const PairConst &K = C.kc;
    KScalD o;
    cxd A, Ap, df, dfp;
    if (K.kmax * R < kSeriesRho) {
        const double r1 = 0.079577471545947667884 * rinv, r2 = r1 * rinv, r3 = r2 * rinv;
        cxd S, Sp;
        horner_d(Ks.cD, R, S, Sp);
        A = r1 * S;
        Ap = r1 * Sp - rinv * A;
        horner_d(Ks.cG, R, S, Sp);
        const cxd dg = r3 * S;
        A = A - dg;
        Ap = Ap - (r3 * Sp - (3.0 * rinv) * dg);
        horner_d(Ks.cF, R, S, Sp);
        df = r3 * S;
        dfp = r3 * Sp - (3.0 * rinv) * df;
        horner_d(Ks.cE, R, S, Sp);
        o.Ge = r2 * S;
        o.Gep = r2 * Sp - (2.0 * rinv) * o.Ge;
        horner_d(Ks.cM, R, S, Sp);
        o.Gm = r2 * S;
        o.Gmp = r2 * Sp - (2.0 * rinv) * o.Gm;
    } else {
        const double r1 = 0.079577471545947667884 * rinv, r2 = r1 * rinv, r3 = r2 * rinv, r4 = r3 * rinv;
        const Media64 m = media64(K, R);
        const cxd ep = {K.eps_re, K.eps_im}, mu = {K.mu_re, K.mu_im};
        const cxd f = m.fa - m.fi, q = m.ta2 * m.ga - m.ti2 * m.gi;
        df = r3 * f;
        dfp = r4 * (q - 3.0 * f);
        A = r1 * m.d - r3 * (m.ga - m.gi);
        Ap = r4 * (f - q);
        const cxd Eg = m.ga - ep * m.gi, Mg = m.ga - mu * m.gi;
        o.Ge = (-r2) * Eg;
        o.Gep = r3 * (2.0 * Eg - (m.ha - ep * m.hi));
        o.Gm = (-r2) * Mg;
        o.Gmp = r3 * (2.0 * Mg - (m.ha - mu * m.hi));
    }
    o.a = C.iw * A;
    o.ap = C.iw * Ap;
    o.d = C.iw * df;
    o.dp = C.iw * dfp;
    return o;
}

// ------------------------------------------------- point-pair adjoint ---
// Adds S1, S2, Hj and Hm of one pair (R = x - y, h = R / |R|) and returns
// d Im F / dR.
__device__ __forceinline__ dvec3 pair_terms(const KScalD &s, dvec3 h, double rinv, cv3 u1, cv3 u2, cv3 vj, cv3 vm,
                                            cv3 &S1, cv3 &S2, cv3 &Hj, cv3 &Hm) {
    const cxd v1 = cdot(vj, h), v2 = cdot(vm, h), w1 = cdot(u1, h), w2 = cdot(u2, h);
    const cxd dv1 = s.d * v1, dv2 = s.d * v2, dw1 = s.d * w1, dw2 = s.d * w2;
    const cv3 xm = ccross(vm, h), xj = ccross(vj, h);
    S1 = S1 + (s.a * vj + dv1 * h + s.Ge * xm);
    S2 = S2 + (s.Gm * xj - (s.a * vm + dv2 * h));
    Hj = Hj + (s.a * u1 + dw1 * h + s.Gm * ccross(h, u2));
    Hm = Hm + (s.Ge * ccross(h, u1) - (s.a * u2 + dw2 * h));
    const cxd al = cdot(u1, vj) - cdot(u2, vm), be = w1 * v1 - w2 * v2;
    const cxd ee = cdot(u1, xm), mm = cdot(u2, xj);
    // transverse part: the derivative of F by h
    const dvec3 w = im3(dw1 * vj) + im3(dv1 * u1) - im3(dw2 * vm) - im3(dv2 * u2) + im3(ccross(s.Ge * u1, vm)) +
                    im3(ccross(s.Gm * u2, vj));
    const double wr = (2.0 * (s.d * be) + s.Ge * ee + s.Gm * mm).im;
    const double gr = (s.ap * al + s.dp * be + s.Gep * ee + s.Gmp * mm).im;
    return rinv * w + (gr - rinv * wr) * h;
}

struct TPt {
    dvec3 x, n, t1, t2;
    double W;
    cxd L[4];
};
struct SPt {
    dvec3 y, t1, t2;
    double W;
    cxd X[4];
};
// NODAL (node-attached tangents): the adjoints of the point's vectors p1, p2
// (test) and vj, vm (trial) themselves, complex and not yet reduced to Im,
// in place of those of the point frame.
struct TGrad {
    dvec3 x, n, t1, t2;
    double W;
    cv3 p1, p2;
};
struct SGrad {
    dvec3 y, t1, t2;
    double W;
    cv3 vj, vm;
};
__device__ inline cv3 czero3() { return {{0, 0}, {0, 0}, {0, 0}}; }
__device__ inline void zero(TGrad &g) {
    g.x = g.n = g.t1 = g.t2 = {0, 0, 0};
    g.W = 0.0;
    g.p1 = g.p2 = czero3();
}
__device__ inline void zero(SGrad &g) {
    g.y = g.t1 = g.t2 = {0, 0, 0};
    g.W = 0.0;
    g.vj = g.vm = czero3();
}

// Node-attached field of the coefficients c (node v, component b at
// c[2 v + b]) at a point with shape functions N: m = sum_k N_k sum_b c_kb t_b,k
// (the nodal tangents, not yet projected on the point's tangent plane).
__device__ inline cv3 nodal_field(const double *__restrict__ frames, const int32_t *t, const double N[6],
                                  const double2 *__restrict__ c) {
    cv3 m = czero3();
    for (int k = 0; k < 6; ++k) {
        const int64_t v = t[k];
        for (int b = 0; b < 2; ++b) {
            const double2 cf = c[2 * v + b];
            m = m + cxd{N[k] * cf.x, N[k] * cf.y} * nodal_tangent(frames, v, b);
        }
    }
    return m;
}

// Reverse of p = m - (m.n) n for the adjoint G of p (Im(G.p) is the
// quantity): adds the normal's part to bn and returns the adjoint of m.
__device__ inline cv3 proj_reverse(cv3 G, cv3 m, dvec3 n, dvec3 &bn) {
    const cxd mn = cdot(m, n), Gn = cdot(G, n);
    bn = bn - im3(Gn * m + mn * G);
    return G - Gn * n;
}

// Node-tangent adjoints of one point: Im(N_k sum_f c_f[kb] G_f) for the
// fields f built from the coefficient vectors c_f (nf of them).
template <int NF>
__device__ inline void nodal_tangent_adjoint(const int32_t *t, const double N[6], const double2 *const c[NF],
                                             const cv3 G[NF], dvec3 gT1[6], dvec3 gT2[6]) {
    for (int k = 0; k < 6; ++k) {
        const int64_t v = t[k];
        cv3 g[2] = {czero3(), czero3()};
        for (int f = 0; f < NF; ++f)
            for (int b = 0; b < 2; ++b) {
                const double2 cf = c[f][2 * v + b];
                g[b] = g[b] + cxd{N[k] * cf.x, N[k] * cf.y} * G[f];
            }
        gT1[k] = im3(g[0]);
        gT2[k] = im3(g[1]);
    }
}

// Adjoints of a test point's p1, p2, n and W for c (u1.S1 + u2.S2) / W.
template <bool NODAL>
__device__ inline void test_adjoint(const TPt &P, cv3 S1, cv3 S2, double c, TGrad &gt) {
    const cv3 p1 = P.L[0] * P.t1 + P.L[1] * P.t2, p2 = P.L[2] * P.t1 + P.L[3] * P.t2;
    const cv3 g1 = ccross(P.n, S1), g2 = ccross(P.n, S2);
    const double cw = c * P.W;
    gt.n = gt.n + cw * im3(ccross(S1, p1) + ccross(S2, p2));
    if constexpr (NODAL) {
        gt.p1 = gt.p1 + cw * g1;
        gt.p2 = gt.p2 + cw * g2;
    } else {
        gt.t1 = gt.t1 + cw * im3(P.L[0] * g1 + P.L[2] * g2);
        gt.t2 = gt.t2 + cw * im3(P.L[1] * g1 + P.L[3] * g2);
    }
    // p.(n x S) = (p x n).S
    gt.W += c * (cdot(p1, g1) + cdot(p2, g2)).im;
}
template <bool NODAL>
__device__ inline void trial_adjoint(const SPt &Q, cv3 Hj, cv3 Hm, double c, SGrad &gs) {
    const double cw = c * Q.W;
    const cv3 vj = Q.X[0] * Q.t1 + Q.X[1] * Q.t2, vm = Q.X[2] * Q.t1 + Q.X[3] * Q.t2;
    if constexpr (NODAL) {
        gs.vj = gs.vj + cw * Hj;
        gs.vm = gs.vm + cw * Hm;
    } else {
        gs.t1 = gs.t1 + cw * im3(Q.X[0] * Hj + Q.X[2] * Hm);
        gs.t2 = gs.t2 + cw * im3(Q.X[1] * Hj + Q.X[3] * Hm);
    }
    gs.W += c * (cdot(vj, Hj) + cdot(vm, Hm)).im;
}

// --------------------------------------------------- per-point fields ---
// fields[i][0..7]: L0..L3 (lambda), [8..15]: X0..X3 (x) at regular point i.
// NODAL: the components in the point frame of the node-attached fields,
// L = (m1.t1, m1.t2, m2.t1, m2.t2) with m1, m2 the fields of lambda's two
// currents, X likewise from x, so that L0 t1 + L1 t2 = P m1 exactly.
// tab[14][nq]: the position (3 reals and a zero), then W u1, W u2, W vj, W vm.
constexpr int kTab = 14;
template <bool NODAL>
__global__ void k_qp_fields(int64_t nt, int64_t n2, const int32_t *__restrict__ tri,
                            const double *__restrict__ qp, const double *__restrict__ frames,
                            const double2 *__restrict__ lam, const double2 *__restrict__ x,
                            double *__restrict__ fields, double2 *__restrict__ tab) {
    const int64_t nq = nt * kQP;
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= nq) return;
    const int64_t e = i / kQP;
    double xi, eta, w, N[6], d1[6], d2[6];
    rule7((int)(i % kQP), xi, eta, w);
    p2_shape(xi, eta, N, d1, d2);
    const dvec3 t1 = {qp[QT1 * nq + i], qp[(QT1 + 1) * nq + i], qp[(QT1 + 2) * nq + i]};
    const dvec3 t2 = {qp[QT2 * nq + i], qp[(QT2 + 1) * nq + i], qp[(QT2 + 2) * nq + i]};
    cxd c[8];
    if constexpr (NODAL) {
        const double2 *cf[4] = {lam, lam + n2, x, x + n2};
        for (int f = 0; f < 4; ++f) {
            const cv3 m = nodal_field(frames, tri + 6 * e, N, cf[f]);
            c[2 * f] = cdot(m, t1);
            c[2 * f + 1] = cdot(m, t2);
        }
    } else {
        for (int k = 0; k < 8; ++k) c[k] = {0.0, 0.0};
        for (int k = 0; k < 6; ++k) {
            const int64_t nd = tri[6 * e + k];
            const double2 v[8] = {lam[2 * nd], lam[2 * nd + 1], lam[n2 + 2 * nd], lam[n2 + 2 * nd + 1],
                                  x[2 * nd], x[2 * nd + 1], x[n2 + 2 * nd], x[n2 + 2 * nd + 1]};
            for (int j = 0; j < 8; ++j) c[j] = c[j] + cxd{N[k] * v[j].x, N[k] * v[j].y};
        }
    }
    for (int k = 0; k < 8; ++k) { fields[16 * i + 2 * k] = c[k].re; fields[16 * i + 2 * k + 1] = c[k].im; }
    const dvec3 nv = {qp[QN * nq + i], qp[(QN + 1) * nq + i], qp[(QN + 2) * nq + i]};
    const double W = qp[QW * nq + i];
    tab[i] = double2{qp[QX * nq + i], qp[(QX + 1) * nq + i]};
    tab[nq + i] = double2{qp[(QX + 2) * nq + i], 0.0};
    for (int f = 0; f < 4; ++f) {
        const cv3 m = W * (c[2 * f] * t1 + c[2 * f + 1] * t2), v = f < 2 ? ccross(m, nv) : m;
        tab[(2 + 3 * f) * nq + i] = double2{v.x.re, v.x.im};
        tab[(3 + 3 * f) * nq + i] = double2{v.y.re, v.y.im};
        tab[(4 + 3 * f) * nq + i] = double2{v.z.re, v.z.im};
    }
}

__device__ inline void load_tpt(const double *qp, const double *fields, int64_t nq, int64_t i, TPt &P) {
    P.x = {qp[QX * nq + i], qp[(QX + 1) * nq + i], qp[(QX + 2) * nq + i]};
    P.W = qp[QW * nq + i];
    P.n = {qp[QN * nq + i], qp[(QN + 1) * nq + i], qp[(QN + 2) * nq + i]};
    P.t1 = {qp[QT1 * nq + i], qp[(QT1 + 1) * nq + i], qp[(QT1 + 2) * nq + i]};
    P.t2 = {qp[QT2 * nq + i], qp[(QT2 + 1) * nq + i], qp[(QT2 + 2) * nq + i]};
    const double *f = fields + 16 * i;
    for (int c = 0; c < 4; ++c) P.L[c] = {f[2 * c], f[2 * c + 1]};
}
__device__ inline void load_spt(const double *qp, const double *fields, int64_t nq, int64_t i, SPt &Q) {
    Q.y = {qp[QX * nq + i], qp[(QX + 1) * nq + i], qp[(QX + 2) * nq + i]};
    Q.W = qp[QW * nq + i];
    Q.t1 = {qp[QT1 * nq + i], qp[(QT1 + 1) * nq + i], qp[(QT1 + 2) * nq + i]};
    Q.t2 = {qp[QT2 * nq + i], qp[(QT2 + 1) * nq + i], qp[(QT2 + 2) * nq + i]};
    const double *f = fields + 16 * i + 8;
    for (int c = 0; c < 4; ++c) Q.X[c] = {f[2 * c], f[2 * c + 1]};
}

// --------------------------------------------------- regular pairs ---
// Point adjoint table qb[i][13]: x(3), W(1), n(3), t1(3), t2(3).
// NODAL, qb[i][31]: x(3), W(1), n(3), then the complex adjoints (re, im per
// component) of p1, p2 (test side) and vj, vm (trial side).
constexpr int kQB = 13;
constexpr int kQBN = 31;
template <bool NODAL> constexpr int qb_stride() { return NODAL ? kQBN : kQB; }

__device__ inline void put_cv3(double *o, cv3 v) {
    o[0] = v.x.re; o[1] = v.x.im; o[2] = v.y.re; o[3] = v.y.im; o[4] = v.z.re; o[5] = v.z.im;
}
__device__ inline cv3 get_cv3(const double *o) { return {{o[0], o[1]}, {o[2], o[3]}, {o[4], o[5]}}; }

// One wavefront per (64 test points, 64 trial points, run of steps): lane l
// holds test point l and meets trial point (l + s) % 64 in step s, whose data
// and sums wait in LDS, so each pair is evaluated once for both sides and no
// sum crosses lanes.  acc[30][nq]: S1, S2 and the position's sum of the test
// point, Hj, Hm and the position's sum of the trial point.
// Bound by FP64 vector instructions (about 500 a pair).  Sphere of 1280
// triangles: 7.3 ms as two passes with one side's adjoints formed pair by pair,
// divisions and a reduction at the end -> 2.0 ms here.
constexpr int kSide = 15;     // sums of one side
constexpr int kShapeTile = 64;

__device__ inline dvec3 tab_pos(double2 a, double2 b) { return {a.x, a.y, b.x}; }
__device__ inline cv3 tab_vec(double2 a, double2 b, double2 c) { return {{a.x, a.y}, {b.x, b.y}, {c.x, c.y}}; }

__global__ __launch_bounds__(64, 2) void k_shape_regular(int64_t nq, int tiles, int steps,
                                                         const double2 *__restrict__ tab,
                                                         const int32_t *__restrict__ tri, ShapeConst C,
                                                         const KernelConst *__restrict__ Kp,
                                                         double *__restrict__ acc) {
    __shared__ double2 s_t[8][kShapeTile], s_a[8][kShapeTile];
    __shared__ int32_t s_f[3][kShapeTile];
    __shared__ KernelConst s_K;
    const int lane = threadIdx.x;
    const int64_t i = (int64_t)blockIdx.y * kShapeTile + lane, j = (int64_t)(blockIdx.x % tiles) * kShapeTile + lane;
    const int s0 = (int)(blockIdx.x / tiles) * steps;
    constexpr int nw = (int)(sizeof(KernelConst) / sizeof(double));
    for (int k = lane; k < nw; k += 64) ((double *)&s_K)[k] = ((const double *)Kp)[k];
    const int64_t ic = i < nq ? i : nq - 1, jc = j < nq ? j : nq - 1;
    int32_t te[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        te[k] = tri[6 * (ic / kQP) + k];
        s_f[k][lane] = j < nq ? tri[6 * (jc / kQP) + k] : -1;
    }
    const dvec3 x = tab_pos(tab[ic], tab[nq + ic]);
    const cv3 u1 = tab_vec(tab[2 * nq + ic], tab[3 * nq + ic], tab[4 * nq + ic]);
    const cv3 u2 = tab_vec(tab[5 * nq + ic], tab[6 * nq + ic], tab[7 * nq + ic]);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        s_t[k][lane] = tab[(k < 2 ? k : 6 + k) * nq + jc];
        s_a[k][lane] = double2{0.0, 0.0};
    }
    cv3 S1 = czero3(), S2 = S1;
    dvec3 gx = {0, 0, 0};
    __syncthreads();
    for (int s = s0; s < s0 + steps; ++s) {
        const int k = (lane + s) % kShapeTile;
        const int32_t f0 = s_f[0][k], f1 = s_f[1][k], f2 = s_f[2][k];
        bool on = i < nq && f0 >= 0;                   // pairs that share a vertex are not regular
#pragma unroll
        for (int c = 0; c < 3; ++c) on = on && te[c] != f0 && te[c] != f1 && te[c] != f2;
        if (on) {
            const dvec3 Rv = x - tab_pos(s_t[0][k], s_t[1][k]);
            const cv3 vj = tab_vec(s_t[2][k], s_t[3][k], s_t[4][k]), vm = tab_vec(s_t[5][k], s_t[6][k], s_t[7][k]);
            const Root64 root = root64(dot(Rv, Rv));
            const double rinv = root.inv;
            const KScalD sc = kernel_scalars_dr(C, s_K, root.r, rinv);
            cv3 Hj = tab_vec(s_a[0][k], s_a[1][k], s_a[2][k]), Hm = tab_vec(s_a[3][k], s_a[4][k], s_a[5][k]);
            const dvec3 g = pair_terms(sc, rinv * Rv, rinv, u1, u2, vj, vm, S1, S2, Hj, Hm);
            gx = gx + g;
            s_a[0][k] = double2{Hj.x.re, Hj.x.im};
            s_a[1][k] = double2{Hj.y.re, Hj.y.im};
            s_a[2][k] = double2{Hj.z.re, Hj.z.im};
            s_a[3][k] = double2{Hm.x.re, Hm.x.im};
            s_a[4][k] = double2{Hm.y.re, Hm.y.im};
            s_a[5][k] = double2{Hm.z.re, Hm.z.im};
            const double2 a6 = s_a[6][k], a7 = s_a[7][k];
            s_a[6][k] = double2{a6.x + g.x, a6.y + g.y};
            s_a[7][k] = double2{a7.x + g.z, 0.0};
        }
        __syncthreads();                               // the next lane's turn at trial point k
    }
    if (i < nq) {
        const double v[kSide] = {S1.x.re, S1.x.im, S1.y.re, S1.y.im, S1.z.re, S1.z.im, S2.x.re, S2.x.im,
                                 S2.y.re, S2.y.im, S2.z.re, S2.z.im, gx.x, gx.y, gx.z};
#pragma unroll
        for (int c = 0; c < kSide; ++c) unsafeAtomicAdd(acc + c * nq + i, v[c]);
    }
    if (j < nq) {
#pragma unroll
        for (int c = 0; c < kSide; ++c)
            unsafeAtomicAdd(acc + (kSide + c) * nq + j, c & 1 ? s_a[c / 2][lane].y : s_a[c / 2][lane].x);
    }
}

// What acc holds at point i, as adjoints of its quantities.
template <bool NODAL>
__device__ inline void regular_adjoint(const double *__restrict__ acc, int64_t nq, int64_t i, const TPt &P,
                                       const SPt &Q, TGrad &gt, SGrad &gs) {
    double v[2 * kSide];
#pragma unroll
    for (int c = 0; c < 2 * kSide; ++c) v[c] = acc[c * nq + i];
    test_adjoint<NODAL>(P, get_cv3(v), get_cv3(v + 6), -1.0, gt);
    trial_adjoint<NODAL>(Q, get_cv3(v + kSide), get_cv3(v + kSide + 6), -1.0, gs);
    gt.x = gt.x - dvec3{v[12], v[13], v[14]};
    gs.y = gs.y + dvec3{v[kSide + 12], v[kSide + 13], v[kSide + 14]};
}

// ------------------------------------------------ single-point terms ---
// The regular pairs' sums (acc) and
// + Im(g^T x)    far field functional, g^T x = sum_q pre W [j.e_perp - j_m.(e x r)]
// + Im(lambda^T b)  right-hand side, sum_q W [-u1.E + u2.H]
// - Im(lambda^T M-part x)  mass, sum_q W [c_eps (L0 X2 + L1 X3) + c_mu (L2 X0 + L3 X1)]
struct SingleArgs {
    dvec3 khat;
    cxd pol[3], ec[3];    // incident polarisation, conj(pol)
    double ka;
    cxd ce, cm;
};

template <bool NODAL>
__global__ __launch_bounds__(256) void k_shape_single(int64_t nt, const double *__restrict__ qp, const double *__restrict__ fields,
                               SingleArgs a, const double *__restrict__ acc, double *__restrict__ qb) {
    const int64_t nq = nt * kQP;
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= nq) return;
    TPt P;
    SPt Q;
    load_tpt(qp, fields, nq, i, P);
    load_spt(qp, fields, nq, i, Q);
    const dvec3 r = a.khat, y = P.x, n = P.n;
    const double W = P.W;
    dvec3 gx = {0, 0, 0}, gn = {0, 0, 0}, gt1 = {0, 0, 0}, gt2 = {0, 0, 0};
    double gW = 0.0;
    // NODAL: complex adjoints of the point's vectors p1, p2, vj, vm
    cv3 gp1 = czero3(), gp2 = czero3(), gvj = czero3(), gvm = czero3();
    {
        TGrad gt;
        SGrad gs;
        zero(gt);
        zero(gs);
        regular_adjoint<NODAL>(acc, nq, i, P, Q, gt, gs);
        gx = gt.x + gs.y;
        gn = gt.n;
        gW = gt.W + gs.W;
        gt1 = gt.t1 + gs.t1;
        gt2 = gt.t2 + gs.t2;
        gp1 = gt.p1;
        gp2 = gt.p2;
        gvj = gs.vj;
        gvm = gs.vm;
    }
    // far field
    {
        double sn, cs;
        sincos(-a.ka * dot(r, y), &sn, &cs);
        const cxd pre = cxd{0.0, a.ka * 0.079577471545947667884} * cxd{cs, sn};
        const cv3 e = {a.ec[0], a.ec[1], a.ec[2]};
        const cxd re = cdot(e, r);
        const cv3 ep = e - re * r;
        const cv3 ex = ccross(e, r);
        const cv3 j = Q.X[0] * P.t1 + Q.X[1] * P.t2, jm = Q.X[2] * P.t1 + Q.X[3] * P.t2;
        const cxd G1 = cdot(j, ep) - cdot(jm, ex);
        const cxd T = pre * cxd{W * G1.re, W * G1.im};
        gx = gx + im3(cxd{0.0, -a.ka} * T * r);
        gW += (pre * G1).im;
        if constexpr (NODAL) {
            gvj = gvj + (cxd{W, 0} * pre) * ep;
            gvm = gvm - (cxd{W, 0} * pre) * ex;
        } else {
            gt1 = gt1 + im3((cxd{W, 0} * pre) * (Q.X[0] * ep - Q.X[2] * ex));
            gt2 = gt2 + im3((cxd{W, 0} * pre) * (Q.X[1] * ep - Q.X[3] * ex));
        }
    }
    // right-hand side
    {
        double sn, cs;
        sincos(a.ka * dot(a.khat, y), &sn, &cs);
        const cxd ph = {cs, sn};
        const cv3 E = {ph * a.pol[0], ph * a.pol[1], ph * a.pol[2]};
        const cv3 H = ccross(a.khat, E);
        const cv3 p1 = P.L[0] * P.t1 + P.L[1] * P.t2, p2 = P.L[2] * P.t1 + P.L[3] * P.t2;
        const cv3 u1 = ccross(p1, n), u2 = ccross(p2, n);
        const cxd V = cdot(u2, H) - cdot(u1, E);
        gW += V.im;
        gx = gx + im3((cxd{0.0, a.ka} * cxd{W * V.re, W * V.im}) * a.khat);
        const cv3 g_u1 = cxd{-W, 0.0} * E, g_u2 = cxd{W, 0.0} * H;
        const cv3 g_p1 = ccross(n, g_u1), g_p2 = ccross(n, g_u2);
        gn = gn + im3(ccross(g_u1, p1) + ccross(g_u2, p2));
        if constexpr (NODAL) {
            gp1 = gp1 + g_p1;
            gp2 = gp2 + g_p2;
        } else {
            gt1 = gt1 + im3(P.L[0] * g_p1 + P.L[2] * g_p2);
            gt2 = gt2 + im3(P.L[1] * g_p1 + P.L[3] * g_p2);
        }
    }
    // mass (p1 . vm = L0 X2 + L1 X3: both are expansions on the same
    // orthonormal pair)
    {
        const cxd m = a.ce * (P.L[0] * Q.X[2] + P.L[1] * Q.X[3]) + a.cm * (P.L[2] * Q.X[0] + P.L[3] * Q.X[1]);
        gW -= m.im;
        if constexpr (NODAL) {
            const cv3 p1 = P.L[0] * P.t1 + P.L[1] * P.t2, p2 = P.L[2] * P.t1 + P.L[3] * P.t2;
            const cv3 vj = Q.X[0] * P.t1 + Q.X[1] * P.t2, vm = Q.X[2] * P.t1 + Q.X[3] * P.t2;
            const cxd we = cxd{-W, 0} * a.ce, wm = cxd{-W, 0} * a.cm;
            gp1 = gp1 + we * vm;
            gvm = gvm + we * p1;
            gp2 = gp2 + wm * vj;
            gvj = gvj + wm * p2;
        }
    }
    constexpr int kS = qb_stride<NODAL>();
    double v[kS];
    v[0] = gx.x; v[1] = gx.y; v[2] = gx.z; v[3] = gW; v[4] = gn.x; v[5] = gn.y; v[6] = gn.z;
    if constexpr (NODAL) {
        put_cv3(v + 7, gp1);
        put_cv3(v + 13, gp2);
        put_cv3(v + 19, gvj);
        put_cv3(v + 25, gvm);
    } else {
        v[7] = gt1.x; v[8] = gt1.y; v[9] = gt1.z; v[10] = gt2.x; v[11] = gt2.y; v[12] = gt2.z;
    }
    double *o = qb + i * kS;
    for (int c = 0; c < kS; ++c) o[c] = v[c];
}

// ------------------------------------------ P2 point: forward + reverse ---
struct P2Fwd {
    dvec3 x, a1, a2, c, n, u1, u2, w1, w2, w3, t1, t2;
    double J, l1, l3;     // |w1|, |w3|
    double N[6], Nxi[6], Neta[6];
};

__device__ inline void p2_forward(const double *__restrict__ xyz, const double *__restrict__ frames,
                                  const int32_t *t, double xi, double eta, P2Fwd &P) {
    p2_shape(xi, eta, P.N, P.Nxi, P.Neta);
    P.x = {0, 0, 0}; P.a1 = {0, 0, 0}; P.a2 = {0, 0, 0}; P.u1 = {0, 0, 0}; P.u2 = {0, 0, 0};
    for (int k = 0; k < 6; ++k) {
        const int64_t v = t[k];
        const dvec3 X = load3(xyz, v);
        P.x = P.x + P.N[k] * X;
        P.a1 = P.a1 + P.Nxi[k] * X;
        P.a2 = P.a2 + P.Neta[k] * X;
        const double *f = frames + 9 * v;
        P.u1 = P.u1 + P.N[k] * dvec3{f[3], f[4], f[5]};
        P.u2 = P.u2 + P.N[k] * dvec3{f[6], f[7], f[8]};
    }
    P.c = cross(P.a1, P.a2);
    P.J = sqrt(dot(P.c, P.c));
    P.n = (1.0 / P.J) * P.c;
    P.w1 = P.u1 - dot(P.n, P.u1) * P.n;
    P.l1 = sqrt(dot(P.w1, P.w1));
    P.t1 = (1.0 / P.l1) * P.w1;
    P.w2 = P.u2 - dot(P.n, P.u2) * P.n;
    P.w3 = P.w2 - dot(P.t1, P.w2) * P.t1;
    P.l3 = sqrt(dot(P.w3, P.w3));
    P.t2 = (1.0 / P.l3) * P.w3;
}

// Adjoints of (x, J, n, t1, t2) -> node positions (gX) and nodal tangents
// (gT1, gT2) of the 6 nodes of the triangle.
__device__ inline void p2_reverse(const P2Fwd &P, dvec3 bx, double bJ, dvec3 bn, dvec3 bt1, dvec3 bt2, dvec3 gX[6],
                                  dvec3 gT1[6], dvec3 gT2[6]) {
    // t2 = w3 / |w3|
    const dvec3 bw3 = (1.0 / P.l3) * (bt2 - dot(bt2, P.t2) * P.t2);
    // w3 = w2 - (t1.w2) t1
    const double s = dot(P.t1, P.w2), bs = dot(bw3, P.t1);
    const dvec3 bw2 = bw3 - bs * P.t1;
    bt1 = bt1 - bs * P.w2 - s * bw3;
    // w2 = u2 - (n.u2) n
    const double nu2 = dot(P.n, P.u2), bwn2 = dot(bw2, P.n);
    const dvec3 bu2 = bw2 - bwn2 * P.n;
    bn = bn - bwn2 * P.u2 - nu2 * bw2;
    // t1 = w1 / |w1|
    const dvec3 bw1 = (1.0 / P.l1) * (bt1 - dot(bt1, P.t1) * P.t1);
    // w1 = u1 - (n.u1) n
    const double nu1 = dot(P.n, P.u1), bwn1 = dot(bw1, P.n);
    const dvec3 bu1 = bw1 - bwn1 * P.n;
    bn = bn - bwn1 * P.u1 - nu1 * bw1;
    // n = c / J, J = |c|
    const dvec3 bc = (1.0 / P.J) * (bn - dot(bn, P.n) * P.n) + bJ * P.n;
    // c = a1 x a2
    const dvec3 ba1 = cross(P.a2, bc), ba2 = cross(bc, P.a1);
    for (int k = 0; k < 6; ++k) {
        gX[k] = P.N[k] * bx + P.Nxi[k] * ba1 + P.Neta[k] * ba2;
        gT1[k] = P.N[k] * bu1;
        gT2[k] = P.N[k] * bu2;
    }
}

__device__ inline void atomic_add3(double *p, dvec3 v) {
    unsafeAtomicAdd(p, v.x);
    unsafeAtomicAdd(p + 1, v.y);
    unsafeAtomicAdd(p + 2, v.z);
}

// Regular points: back through the P2 map and frame of their triangle.
// nodeb[v][9]: position (3), nodal t1 (3), nodal t2 (3) adjoints.
// NODAL: back through the projections p = m - (m.n) n of the four
// node-attached fields to the normal and the nodal tangents; the point
// frame does not enter.
template <bool NODAL>
__global__ __launch_bounds__(256) void k_qp_backprop(int64_t nt, int64_t n2, const double *__restrict__ xyz,
                              const double *__restrict__ frames, const int32_t *__restrict__ tri,
                              const double2 *__restrict__ lam, const double2 *__restrict__ x,
                              const double *__restrict__ qb, double *__restrict__ nodeb) {
    const int64_t nq = nt * kQP;
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= nq) return;
    const int64_t e = i / kQP;
    double xi, eta, w;
    rule7((int)(i % kQP), xi, eta, w);
    P2Fwd P;
    p2_forward(xyz, frames, tri + 6 * e, xi, eta, P);
    constexpr int kS = qb_stride<NODAL>();
    const double *b = qb + i * kS;
    dvec3 gX[6], gT1[6], gT2[6];
    if constexpr (NODAL) {
        const int32_t *t = tri + 6 * e;
        const double2 *c[4] = {lam, lam + n2, x, x + n2};
        dvec3 bn = {b[4], b[5], b[6]};
        cv3 gm[4];
        for (int f = 0; f < 4; ++f)
            gm[f] = proj_reverse(get_cv3(b + 7 + 6 * f), nodal_field(frames, t, P.N, c[f]), P.n, bn);
        p2_reverse(P, {b[0], b[1], b[2]}, w * b[3], bn, {0, 0, 0}, {0, 0, 0}, gX, gT1, gT2);
        nodal_tangent_adjoint<4>(t, P.N, c, gm, gT1, gT2);
    } else {
        p2_reverse(P, {b[0], b[1], b[2]}, w * b[3], {b[4], b[5], b[6]}, {b[7], b[8], b[9]}, {b[10], b[11], b[12]},
                   gX, gT1, gT2);
    }
    for (int k = 0; k < 6; ++k) {
        double *o = nodeb + 9 * (int64_t)tri[6 * e + k];
        atomic_add3(o, gX[k]);
        atomic_add3(o + 3, gT1[k]);
        atomic_add3(o + 6, gT2[k]);
    }
}

// ------------------------------------------------- singular pairs ---
// One wavefront per (coincident / common-edge / common-vertex pair, two
// regions): the Sauter-Schwab points of the fill, one per lane and batch.  Every
// field of a triangle is a polynomial in LDS (as node data in registers they
// spilled 436 scalars): position, nodal tangents and current coefficients;
// NODAL: position and the node-attached vectors m of two currents.  A point's
// geometry is formed twice, for the pair and again for its reverse, to end its
// registers' lives in between.  The adjoints of the six nodes are summed over
// the points by the matrix cores: a 4x4x4 instruction whose first factor has
// ones in row r alone adds a lane value over the four groups of 16 lanes into
// row r, so four columns share one register of sums and nothing crosses lanes
// until the end (before: every batch through LDS and 64 reads a column).
// Columns per side: 6 x 3 positions, 6 x 3 of each tangent; NODAL: 6 x 12 of the
// adjoints of m, which the tangents' follow from at the end.
// Bound by FP64 vector instructions at two wavefronts per SIMD.  1280 triangles:
// 3.80 -> 1.63 ms, node-attached tangents about 2.1 (one wavefront per SIMD, nothing
// spilled: 2.23 and 2.15; all of a point kept live: 108 spills in place of 46).
struct ShapeSsqArgs {
    int64_t n2, npairs;
    const int32_t *pairs, *tri;
    const double *xyz, *frames;
    const double2 *lam, *x;
    int order;
    int64_t np;             // table points
    const double *tab;
    const KernelConst *K;
    ShapeConst C;
    double *nodeb;
};

// What was read from LDS before is read again behind this (no instruction).
__device__ __forceinline__ void reload_lds() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

// Position, normal, metric and first derivatives of a triangle's polynomials
// (F fields, coefficient k of field f at co[F k + f]).
struct SsqGeom {
    dvec3 x, a1, a2, n;
    double J, Ji;
};
template <int F>
__device__ __forceinline__ SsqGeom ssq_geom(const double *co, double xi, double eta) {
    double v[3], d1[3], d2[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double c3 = co[3 * F + d], c4 = co[4 * F + d], c5 = co[5 * F + d];
        const double t = fma(c3, xi, fma(c4, eta, co[F + d])), s = fma(c5, eta, co[2 * F + d]);
        v[d] = fma(xi, t, fma(eta, s, co[d]));
        d1[d] = fma(c3, xi, t);
        d2[d] = fma(c4, xi, fma(c5, eta, s));
    }
    SsqGeom g;
    g.x = {v[0], v[1], v[2]};
    g.a1 = {d1[0], d1[1], d1[2]};
    g.a2 = {d2[0], d2[1], d2[2]};
    const dvec3 c = cross(g.a1, g.a2);
    const Root64 root = root64(dot(c, c));
    g.Ji = root.inv;
    g.J = root.r;
    g.n = g.Ji * c;
    return g;
}
template <int F>
__device__ __forceinline__ double ssq_field(const double *co, int f, double xi, double eta) {
    const double t = fma(co[3 * F + f], xi, fma(co[4 * F + f], eta, co[F + f])), s = fma(co[5 * F + f], eta, co[2 * F + f]);
    return fma(xi, t, fma(eta, s, co[f]));
}
template <int F>
__device__ __forceinline__ dvec3 ssq_vec(const double *co, int f, double xi, double eta) {
    return {ssq_field<F>(co, f, xi, eta), ssq_field<F>(co, f + 1, xi, eta), ssq_field<F>(co, f + 2, xi, eta)};
}
template <int F>
__device__ __forceinline__ cv3 ssq_cvec(const double *co, int f, double xi, double eta) {
    const dvec3 a = {ssq_field<F>(co, f, xi, eta), ssq_field<F>(co, f + 2, xi, eta), ssq_field<F>(co, f + 4, xi, eta)};
    const dvec3 b = {ssq_field<F>(co, f + 1, xi, eta), ssq_field<F>(co, f + 3, xi, eta),
                     ssq_field<F>(co, f + 5, xi, eta)};
    return {{a.x, b.x}, {a.y, b.y}, {a.z, b.z}};
}
// the Gram-Schmidt frame of a point from the nodal tangents' fields 3 .. 8
struct SsqFrame {
    dvec3 u1, u2, t1, t2, w2;
    double l1i, l3i;
};
template <int F>
__device__ __forceinline__ SsqFrame ssq_frame(const double *co, double xi, double eta, dvec3 n) {
    SsqFrame f;
    f.u1 = ssq_vec<F>(co, 3, xi, eta);
    f.u2 = ssq_vec<F>(co, 6, xi, eta);
    const dvec3 w1 = f.u1 - dot(n, f.u1) * n;
    f.l1i = root64(dot(w1, w1)).inv;
    f.t1 = f.l1i * w1;
    f.w2 = f.u2 - dot(n, f.u2) * n;
    const dvec3 w3 = f.w2 - dot(f.t1, f.w2) * f.t1;
    f.l3i = root64(dot(w3, w3)).inv;
    f.t2 = f.l3i * w3;
    return f;
}

// What the pair leaves to one side's reverse: the adjoints of position and
// metric, and c S1, c S2 (test side) or c Hj, c Hm (trial side).
struct SideAdj {
    dvec3 bx;
    double bJ;
    cv3 g1, g2;
};

// Back through the point's vectors, map and frame; put(column, value).
template <bool TEST, bool NODAL, int F, typename PUT>
__device__ __forceinline__ void ssq_reverse(const double *co, double xi, double eta, const SideAdj &a, PUT put) {
    const SsqGeom g = ssq_geom<F>(co, xi, eta);
    double N[6], Nxi[6], Neta[6];
    p2_shape(xi, eta, N, Nxi, Neta);
    dvec3 bn = {0, 0, 0};
    // adjoints of the side's two vectors; u = p x n on the test side
    cv3 G1 = a.g1, G2 = a.g2;
    if constexpr (TEST) {
        G1 = ccross(g.n, a.g1);
        G2 = ccross(g.n, a.g2);
    }
    if constexpr (NODAL) {
#pragma unroll
        for (int f = 0; f < 2; ++f) {
            reload_lds();
            const cv3 m = ssq_cvec<F>(co, 3 + 6 * f, xi, eta);
            if constexpr (TEST) bn = bn + im3(ccross(f ? a.g2 : a.g1, m - cdot(m, g.n) * g.n));
            const cv3 gm = proj_reverse(f ? G2 : G1, m, g.n, bn);
            const double v[6] = {gm.x.re, gm.x.im, gm.y.re, gm.y.im, gm.z.re, gm.z.im};
#pragma unroll
            for (int k = 0; k < 6; ++k)
#pragma unroll
                for (int d = 0; d < 6; ++d) put(18 + 12 * k + 6 * f + d, N[k] * v[d]);
        }
    } else {
        reload_lds();
        const SsqFrame fr = ssq_frame<F>(co, xi, eta, g.n);
        reload_lds();
        cxd L[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            L[k] = {ssq_field<F>(co, 9 + 2 * k, xi, eta), ssq_field<F>(co, 10 + 2 * k, xi, eta)};
        if constexpr (TEST)
            bn = im3(ccross(a.g1, L[0] * fr.t1 + L[1] * fr.t2) + ccross(a.g2, L[2] * fr.t1 + L[3] * fr.t2));
        const dvec3 b1 = im3(L[0] * G1 + L[2] * G2), b2 = im3(L[1] * G1 + L[3] * G2);
        // t2 = w3 / |w3|, w3 = w2 - (t1.w2) t1, w2 = u2 - (n.u2) n
        const dvec3 bw3 = fr.l3i * (b2 - dot(b2, fr.t2) * fr.t2);
        const double s = dot(fr.t1, fr.w2), bs = dot(bw3, fr.t1);
        const dvec3 bw2 = bw3 - bs * fr.t1;
        const dvec3 bt1 = b1 - bs * fr.w2 - s * bw3;
        const double bwn2 = dot(bw2, g.n);
        const dvec3 bu2 = bw2 - bwn2 * g.n;
        bn = bn - bwn2 * fr.u2 - dot(g.n, fr.u2) * bw2;
        // t1 = w1 / |w1|, w1 = u1 - (n.u1) n
        const dvec3 bw1 = fr.l1i * (bt1 - dot(bt1, fr.t1) * fr.t1);
        const double bwn1 = dot(bw1, g.n);
        const dvec3 bu1 = bw1 - bwn1 * g.n;
        bn = bn - bwn1 * fr.u1 - dot(g.n, fr.u1) * bw1;
        const double v[6] = {bu1.x, bu1.y, bu1.z, bu2.x, bu2.y, bu2.z};
#pragma unroll
        for (int k = 0; k < 6; ++k)
#pragma unroll
            for (int d = 0; d < 6; ++d) put(18 + 6 * k + d, N[k] * v[d]);
    }
    // n = c / J, J = |c|, c = a1 x a2
    const dvec3 bc = g.Ji * (bn - dot(bn, g.n) * g.n) + a.bJ * g.n;
    const dvec3 ba1 = cross(g.a2, bc), ba2 = cross(bc, g.a1);
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const dvec3 v = N[k] * a.bx + Nxi[k] * ba1 + Neta[k] * ba2;
        put(3 * k, v.x);
        put(3 * k + 1, v.y);
        put(3 * k + 2, v.z);
    }
}

// The polynomials of both triangles of a pair (fields of a side: NODAL 15, else 17)
template <bool NODAL, int F>
__device__ inline void ssq_polynomials(const ShapeSsqArgs &a, const int32_t *te, const int32_t *tf,
                                       double (*s_co)[6 * F]) {
    for (int it = threadIdx.x; it < 2 * F; it += 64) {
        const int side = it / F, d = it % F;
        const int32_t *t = side ? tf : te;
        const double2 *c = side ? a.x : a.lam;
        double v[6];
        for (int q = 0; q < 6; ++q) {
            const int64_t nd = t[q];
            if (d < 3) {
                v[q] = a.xyz[3 * nd + d] - a.xyz[3 * (int64_t)te[0] + d];
            } else if (NODAL) {
                // m_f = c_f0 t1 + c_f1 t2, component d' (re, im)
                const int fld = (d - 3) / 6, comp = (d - 3) % 6 / 2, im = (d - 3) % 2;
                const double2 c0 = c[fld * a.n2 + 2 * nd], c1 = c[fld * a.n2 + 2 * nd + 1];
                const double *fr = a.frames + 9 * nd;
                v[q] = (im ? c0.y : c0.x) * fr[3 + comp] + (im ? c1.y : c1.x) * fr[6 + comp];
            } else if (d < 9) {
                v[q] = a.frames[9 * nd + d];
            } else {
                const int k = (d - 9) / 2;
                const double2 w = c[(k / 2) * a.n2 + 2 * nd + k % 2];
                v[q] = d % 2 ? w.x : w.y;
            }
        }
#pragma unroll
        for (int k = 0; k < 6; ++k) s_co[side][F * k + d] = p2_coef(k, v);
    }
}
// The two vectors of a side's point (p1, p2 or vj, vm).
template <bool NODAL, int F>
__device__ __forceinline__ void ssq_vectors(const double *co, double xi, double eta, dvec3 n, cv3 &p, cv3 &q) {
    if constexpr (NODAL) {
        p = ssq_cvec<F>(co, 3, xi, eta);
        q = ssq_cvec<F>(co, 9, xi, eta);
        p = p - cdot(p, n) * n;
        q = q - cdot(q, n) * n;
    } else {
        cxd L[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            L[k] = {ssq_field<F>(co, 9 + 2 * k, xi, eta), ssq_field<F>(co, 10 + 2 * k, xi, eta)};
        const SsqFrame fr = ssq_frame<F>(co, xi, eta, n);
        p = L[0] * fr.t1 + L[1] * fr.t2;
        q = L[2] * fr.t1 + L[3] * fr.t2;
    }
}

template <bool NODAL>
__global__ __launch_bounds__(64, 2) void k_shape_ssq(ShapeSsqArgs a) {
    constexpr int F = NODAL ? 15 : 17;                 // fields of a triangle
    constexpr int NCOL = NODAL ? 90 : 54, NACC = (NCOL + 3) / 4;
    __shared__ double s_co[2][6 * F];
    __shared__ KernelConst s_K;
    __shared__ double s_col[2][4 * NACC];
    const int lane = threadIdx.x;
    const int64_t pid = blockIdx.x % a.npairs;
    const int part = (int)(blockIdx.x / a.npairs);
    const int32_t e = a.pairs[4 * pid], f = a.pairs[4 * pid + 1];
    const int cls = a.pairs[4 * pid + 2], code = a.pairs[4 * pid + 3];
    const int nreg = cls == 3 ? 6 : (cls == 2 ? 5 : 2);
    if (2 * part >= nreg) return;
    const int32_t *te = a.tri + 6 * (int64_t)e, *tf = a.tri + 6 * (int64_t)f;
    constexpr int nw = (int)(sizeof(KernelConst) / sizeof(double));
    for (int k = lane; k < nw; k += 64) ((double *)&s_K)[k] = ((const double *)a.K)[k];
    ssq_polynomials<NODAL, F>(a, te, tf, s_co);
    __syncthreads();
    double accT[NACC], accS[NACC], one[4];
#pragma unroll
    for (int k = 0; k < NACC; ++k) accT[k] = accS[k] = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) one[k] = lane % 4 == k ? 1.0 : 0.0;
    const int64_t n4 = (int64_t)a.order * a.order * a.order * a.order, r0 = table_region(cls);
    const int64_t p0 = (r0 + 2 * part) * n4, p1 = (r0 + min(2 * part + 2, nreg)) * n4;
    for (int64_t base = p0; base < p1; base += 64) {
        const int64_t id = base + lane < p1 ? base + lane : p1 - 1;
        const double *q = a.tab + id;
        const double wg = base + lane < p1 ? fabs(q[4 * a.np]) : 0.0;
        double xe, ye, xf, yf;
        ss_local(code & 63, q[0], q[a.np], xe, ye);
        ss_local(code >> 6, q[2 * a.np], q[3 * a.np], xf, yf);
        SideAdj aT, aS;
        {
            const SsqGeom X = ssq_geom<F>(s_co[0], xe, ye), Y = ssq_geom<F>(s_co[1], xf, yf);
            const dvec3 Rv = X.x - Y.x;
            const Root64 root = root64(dot(Rv, Rv));
            const double rinv = root.inv, c = -wg * X.J * Y.J;
            const KScalD sc = kernel_scalars_dr(a.C, s_K, root.r, rinv);
            cv3 u1, u2, vj, vm;
            reload_lds();
            ssq_vectors<NODAL, F>(s_co[0], xe, ye, X.n, u1, u2);
            reload_lds();
            ssq_vectors<NODAL, F>(s_co[1], xf, yf, Y.n, vj, vm);
            u1 = ccross(u1, X.n);
            u2 = ccross(u2, X.n);
            cv3 S1 = czero3(), S2 = S1, Hj = S1, Hm = S1;
            aT.bx = c * pair_terms(sc, rinv * Rv, rinv, u1, u2, vj, vm, S1, S2, Hj, Hm);
            aS.bx = dvec3{0, 0, 0} - aT.bx;
            const double Fi = -wg * (cdot(u1, S1) + cdot(u2, S2)).im;
            aT.bJ = Y.J * Fi;
            aS.bJ = X.J * Fi;
            aT.g1 = c * S1;
            aT.g2 = c * S2;
            aS.g1 = c * Hj;
            aS.g2 = c * Hm;
        }
        reload_lds();                                  // the geometry is formed anew
        ssq_reverse<true, NODAL, F>(s_co[0], xe, ye, aT, [&](int k, double v) {
            accT[k / 4] = __builtin_amdgcn_mfma_f64_4x4x4f64(one[k % 4], v, accT[k / 4], 0, 0, 0);
        });
        reload_lds();
        ssq_reverse<false, NODAL, F>(s_co[1], xf, yf, aS, [&](int k, double v) {
            accS[k / 4] = __builtin_amdgcn_mfma_f64_4x4x4f64(one[k % 4], v, accS[k / 4], 0, 0, 0);
        });
    }
    // row r of register k: column 4 k + r in 16 parts
#pragma unroll
    for (int k = 0; k < NACC; ++k) {
        const double t = rsum16(accT[k]), s = rsum16(accS[k]);
        if (lane % 16 == 0) {
            s_col[0][4 * k + lane / 16] = t;
            s_col[1][4 * k + lane / 16] = s;
        }
    }
    __syncthreads();
    for (int it = lane; it < 108; it += 64) {
        const int side = it / 54, k = it % 54 / 9, comp = it % 9;
        const double *c = s_col[side];
        const int64_t nd = (side ? tf : te)[k];
        double v;
        if (comp < 3) {
            v = c[3 * k + comp];
        } else if constexpr (NODAL) {
            // Im of the current's coefficient times the adjoint of m
            const int b = comp / 3 - 1, d = comp % 3;
            const double2 *cf = side ? a.x : a.lam;
            v = 0.0;
            for (int fld = 0; fld < 2; ++fld) {
                const double2 w = cf[fld * a.n2 + 2 * nd + b];
                const double *g = c + 18 + 12 * k + 6 * fld + 2 * d;
                v += w.x * g[1] + w.y * g[0];
            }
        } else {
            v = c[18 + 6 * k + comp - 3];
        }
        unsafeAtomicAdd(&a.nodeb[9 * nd + comp], v);
    }
}

// ------------------------------------------ lambda^T (dZ/deps) x ---
// The same pairs with the derivatives' scalars: one complex sum, no operator.
// 1280 triangles: 5.4 ms for the fill of dZ/deps, its product and their buffers
// -> 1.5 ms here (the gradient 18.8 -> 14.8 ms, node-attached tangents 24.6 ->
// 15.3).
__device__ __forceinline__ cxd pair_form(const KScal<double> &s, cxd iw, dvec3 h, cv3 u1, cv3 u2, cv3 vj, cv3 vm) {
    const cxd al = cdot(u1, vj) - cdot(u2, vm);
    const cxd be = cdot(u1, h) * cdot(vj, h) - cdot(u2, h) * cdot(vm, h);
    return iw * ((s.D0 - s.dg) * al + s.df * be) + s.Ge * cdot(u1, ccross(vm, h)) + s.Gm * cdot(u2, ccross(vj, h));
}

constexpr int kFormSlots = 256;    // partial sums: a wavefront adds to slot block % kFormSlots
__device__ inline void form_add(double2 *slots, cxd v) {
    const double re = wsum_all(v.re), im = wsum_all(v.im);
    if (threadIdx.x == 0) {
        double2 *o = slots + (blockIdx.x + blockIdx.y * (int64_t)gridDim.x) % kFormSlots;
        unsafeAtomicAdd(&o->x, re);
        unsafeAtomicAdd(&o->y, im);
    }
}

// One wavefront per (64 test points, 64 trial points): a test point per lane,
// the trial points in turn; the first tile adds the points' mass terms.
__global__ __launch_bounds__(64, 4) void k_deps_regular(int64_t nq, const double2 *__restrict__ tab,
                                                     const double *__restrict__ qp,
                                                     const double *__restrict__ fields,
                                                     const int32_t *__restrict__ tri, ShapeConst C, cxd ce, cxd cm,
                                                     const KernelConst *__restrict__ Kp,
                                                     double2 *__restrict__ slots) {
    __shared__ double2 s_t[8][kShapeTile];
    __shared__ int32_t s_f[3][kShapeTile];
    __shared__ KernelConst s_K;
    const int lane = threadIdx.x;
    const int64_t i = (int64_t)blockIdx.y * kShapeTile + lane, j0 = (int64_t)blockIdx.x * kShapeTile;
    const int64_t ic = i < nq ? i : nq - 1, jc = j0 + lane < nq ? j0 + lane : nq - 1;
    const int nj = (int)(nq - j0 < kShapeTile ? nq - j0 : kShapeTile);
    constexpr int nw = (int)(sizeof(KernelConst) / sizeof(double));
    for (int k = lane; k < nw; k += 64) ((double *)&s_K)[k] = ((const double *)Kp)[k];
    int32_t te[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        te[k] = tri[6 * (ic / kQP) + k];
        s_f[k][lane] = tri[6 * (jc / kQP) + k];
    }
    const dvec3 x = tab_pos(tab[ic], tab[nq + ic]);
    const cv3 u1 = tab_vec(tab[2 * nq + ic], tab[3 * nq + ic], tab[4 * nq + ic]);
    const cv3 u2 = tab_vec(tab[5 * nq + ic], tab[6 * nq + ic], tab[7 * nq + ic]);
#pragma unroll
    for (int k = 0; k < 8; ++k) s_t[k][lane] = tab[(k < 2 ? k : 6 + k) * nq + jc];
    __syncthreads();
    cxd sum = {0.0, 0.0};
    for (int k = 0; k < nj; ++k) {
        reload_lds();                                  // the series' coefficients stay in LDS
        bool on = i < nq;                              // pairs that share a vertex are not regular
#pragma unroll
        for (int c = 0; c < 3; ++c) on = on && te[c] != s_f[0][k] && te[c] != s_f[1][k] && te[c] != s_f[2][k];
        if (on) {
            const dvec3 Rv = x - tab_pos(s_t[0][k], s_t[1][k]);
            const cv3 vj = tab_vec(s_t[2][k], s_t[3][k], s_t[4][k]), vm = tab_vec(s_t[5][k], s_t[6][k], s_t[7][k]);
            const Root64 root = root64(dot(Rv, Rv));
            sum = sum + pair_form(kernel_scalars_deps(s_K, root.r, root.inv), C.iw, root.inv * Rv, u1, u2, vj, vm);
        }
    }
    if (blockIdx.x == 0 && i < nq) {
        const double *f = fields + 16 * i;
        cxd v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = {f[2 * k], f[2 * k + 1]};
        sum = sum + qp[QW * nq + i] * (ce * (v[0] * v[6] + v[1] * v[7]) + cm * (v[2] * v[4] + v[3] * v[5]));
    }
    form_add(slots, sum);
}

template <bool NODAL>
__global__ __launch_bounds__(64, 3) void k_deps_ssq(ShapeSsqArgs a, double2 *__restrict__ slots) {
    constexpr int F = NODAL ? 15 : 17;
    __shared__ double s_co[2][6 * F];
    __shared__ KernelConst s_K;
    const int lane = threadIdx.x;
    const int64_t pid = blockIdx.x % a.npairs;
    const int part = (int)(blockIdx.x / a.npairs);
    const int32_t e = a.pairs[4 * pid], f = a.pairs[4 * pid + 1];
    const int cls = a.pairs[4 * pid + 2], code = a.pairs[4 * pid + 3];
    const int nreg = cls == 3 ? 6 : (cls == 2 ? 5 : 2);
    if (2 * part >= nreg) return;
    constexpr int nw = (int)(sizeof(KernelConst) / sizeof(double));
    for (int k = lane; k < nw; k += 64) ((double *)&s_K)[k] = ((const double *)a.K)[k];
    ssq_polynomials<NODAL, F>(a, a.tri + 6 * (int64_t)e, a.tri + 6 * (int64_t)f, s_co);
    __syncthreads();
    const int64_t n4 = (int64_t)a.order * a.order * a.order * a.order, r0 = table_region(cls);
    const int64_t p1 = (r0 + min(2 * part + 2, nreg)) * n4;
    cxd sum = {0.0, 0.0};
    for (int64_t id = (r0 + 2 * part) * n4 + lane; id < p1; id += 64) {
        reload_lds();                                  // no coefficient stays in a register over the points
        const double *q = a.tab + id;
        double xe, ye, xf, yf;
        ss_local(code & 63, q[0], q[a.np], xe, ye);
        ss_local(code >> 6, q[2 * a.np], q[3 * a.np], xf, yf);
        const SsqGeom X = ssq_geom<F>(s_co[0], xe, ye), Y = ssq_geom<F>(s_co[1], xf, yf);
        const dvec3 Rv = X.x - Y.x;
        const Root64 root = root64(dot(Rv, Rv));
        const double rinv = root.inv, w = fabs(q[4 * a.np]) * X.J * Y.J;
        const KScal<double> sc = kernel_scalars_deps(s_K, root.r, rinv);
        cv3 u1, u2, vj, vm;
        reload_lds();
        ssq_vectors<NODAL, F>(s_co[0], xe, ye, X.n, u1, u2);
        reload_lds();
        ssq_vectors<NODAL, F>(s_co[1], xf, yf, Y.n, vj, vm);
        sum = sum + w * pair_form(sc, a.C.iw, rinv * Rv, ccross(u1, X.n),
                                  ccross(u2, X.n), vj, vm);
    }
    form_add(slots, sum);
}

__global__ __launch_bounds__(64) void k_form_sum(const double2 *__restrict__ slots, double2 *__restrict__ out) {
    cxd v = {0.0, 0.0};
    for (int k = threadIdx.x; k < kFormSlots; k += 64) v = v + cxd{slots[k].x, slots[k].y};
    const double re = wsum_all(v.re), im = wsum_all(v.im);
    if (threadIdx.x == 0) *out = double2{re, im};
}

// -------------------------------------------------- nodal frames ---
// Tangents of triangle t at its local node k after the cyclic re-indexing
// that puts the node at the origin (vertex) or at (1/2, 0) (mid-edge node).
__device__ inline void node_tangents(int32_t k, const int32_t *t, const double *X, dvec3 &a1, dvec3 &a2) {
    if (k < 3) {
        const int kn = (k + 1) % 3, kp = (k + 2) % 3;
        a1 = -3.0 * load3(X, t[k]) + 4.0 * load3(X, t[3 + k]) - load3(X, t[kn]);
        a2 = -3.0 * load3(X, t[k]) + 4.0 * load3(X, t[3 + kp]) - load3(X, t[kp]);
    } else {
        const int aa = k - 3, b = (aa + 1) % 3, c = (aa + 2) % 3;
        a1 = load3(X, t[b]) - load3(X, t[aa]);
        a2 = 2.0 * (load3(X, t[3 + b]) + load3(X, t[3 + c]) - load3(X, t[3 + aa])) - load3(X, t[aa]) -
             load3(X, t[c]);
    }
}

// Back through t1 = (ref x n)/|ref x n|, t2 = n x t1 (reference vector held
// fixed), n = S/|S|, S = sum over incident triangles of (a1 x a2)/(g11 g22).
__global__ void k_frames_backprop(int64_t nn, const double *__restrict__ xyz, const int32_t *__restrict__ tri,
                                  const int32_t *__restrict__ inc_ptr, const int32_t *__restrict__ inc,
                                  const double *__restrict__ nodeb_t, double *__restrict__ nodeb_x) {
    const int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (v >= nn) return;
    dvec3 S = {0, 0, 0};
    for (int32_t s = inc_ptr[v]; s < inc_ptr[v + 1]; ++s) {
        dvec3 a1, a2;
        node_tangents(inc[s] & 7, tri + 6 * (inc[s] >> 3), xyz, a1, a2);
        S = S + (1.0 / (dot(a1, a1) * dot(a2, a2))) * cross(a1, a2);
    }
    const double ls = sqrt(dot(S, S));
    const dvec3 n = (1.0 / ls) * S;
    const dvec3 ref = fabs(n.z) > 0.9 ? dvec3{1.0, 0.0, 0.0} : dvec3{0.0, 0.0, 1.0};
    const dvec3 wv = cross(ref, n);
    const double lw = sqrt(dot(wv, wv));
    const dvec3 t1 = (1.0 / lw) * wv;
    const double *b = nodeb_t + 9 * v;
    const dvec3 bt1 = {b[3], b[4], b[5]}, bt2 = {b[6], b[7], b[8]};
    // t2 = n x t1
    dvec3 bn = cross(t1, bt2);
    const dvec3 bt1s = bt1 + cross(bt2, n);
    // t1 = w / |w|, w = ref x n
    const dvec3 bw = (1.0 / lw) * (bt1s - dot(bt1s, t1) * t1);
    bn = bn + cross(bw, ref);
    // n = S / |S|
    const dvec3 bS = (1.0 / ls) * (bn - dot(bn, n) * n);
    for (int32_t s = inc_ptr[v]; s < inc_ptr[v + 1]; ++s) {
        const int32_t k = inc[s] & 7;
        const int32_t *t = tri + 6 * (inc[s] >> 3);
        dvec3 a1, a2;
        node_tangents(k, t, xyz, a1, a2);
        const double g11 = dot(a1, a1), g22 = dot(a2, a2), D = g11 * g22;
        const dvec3 c = cross(a1, a2);
        const dvec3 bc = (1.0 / D) * bS;
        const double q = dot(bS, c) / (D * D);
        const dvec3 ba1 = cross(a2, bc) - (2.0 * q * g22) * a1;
        const dvec3 ba2 = cross(bc, a1) - (2.0 * q * g11) * a2;
        if (k < 3) {
            const int kn = (k + 1) % 3, kp = (k + 2) % 3;
            atomic_add3(nodeb_x + 9 * (int64_t)t[k], -3.0 * (ba1 + ba2));
            atomic_add3(nodeb_x + 9 * (int64_t)t[3 + k], 4.0 * ba1);
            atomic_add3(nodeb_x + 9 * (int64_t)t[kn], -1.0 * ba1);
            atomic_add3(nodeb_x + 9 * (int64_t)t[3 + kp], 4.0 * ba2);
            atomic_add3(nodeb_x + 9 * (int64_t)t[kp], -1.0 * ba2);
        } else {
            const int aa = k - 3, bb = (aa + 1) % 3, cc = (aa + 2) % 3;
            atomic_add3(nodeb_x + 9 * (int64_t)t[bb], ba1);
            atomic_add3(nodeb_x + 9 * (int64_t)t[aa], -1.0 * (ba1 + ba2));
            atomic_add3(nodeb_x + 9 * (int64_t)t[3 + bb], 2.0 * ba2);
            atomic_add3(nodeb_x + 9 * (int64_t)t[3 + cc], 2.0 * ba2);
            atomic_add3(nodeb_x + 9 * (int64_t)t[3 + aa], -2.0 * ba2);
            atomic_add3(nodeb_x + 9 * (int64_t)t[cc], -1.0 * ba2);
        }
    }
}

// d sigma / d delta_v along the displacement direction of node v (dir[v],
// or the nodal normal when dir is null), and the full position gradient
__global__ void k_shape_out(int64_t nn, double scale, const double *__restrict__ frames,
                            const double *__restrict__ dir, const double *__restrict__ nodeb_x, double *dnode,
                            double *dx) {
    const int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (v >= nn) return;
    const double *b = nodeb_x + 9 * v, *nv = dir ? dir + 3 * v : frames + 9 * v;
    if (dnode) dnode[v] = scale * (b[0] * nv[0] + b[1] * nv[1] + b[2] * nv[2]);
    if (dx) for (int c = 0; c < 3; ++c) dx[3 * v + c] = scale * b[c];
}

// --------------------------------------------------------------- host ---
static ShapeConst shape_const(const mbem_op *op) {
    ShapeConst C;
    C.kc = pair_const(op->ka, op->ki, op->eps_i, op->mu_i);
    C.iw = {op->iw.x, op->iw.y};
    return C;
}

// The singular pairs' arguments but for the point table.
static ShapeSsqArgs ssq_args(const mbem_op *op, const double2 *x, const double2 *lam) {
    const mbem_mesh *m = op->mesh;
    ShapeSsqArgs a{};
    a.n2 = op->n2;
    a.npairs = m->n_spairs;
    a.pairs = m->d_spairs;
    a.tri = m->d_tri;
    a.xyz = m->d_xyz;
    a.frames = m->d_frames;
    a.lam = lam;
    a.x = x;
    a.order = op->p.ssq_order > 0 ? op->p.ssq_order : 4;
    a.K = op->d_kconst;
    a.C = shape_const(op);
    return a;
}

static void launch_fields(const mbem_op *op, const double2 *x, const double2 *lam, double *fields, double2 *tab,
                          hipStream_t s) {
    const mbem_mesh *m = op->mesh;
    const dim3 grid((unsigned)((m->nt * kQP + 255) / 256));
    auto k = op->p.frame == MBEM_FRAME_NODAL ? k_qp_fields<true> : k_qp_fields<false>;
    hipLaunchKernelGGL(k, grid, dim3(256), 0, s, m->nt, op->n2, m->d_tri, m->d_qp, m->d_frames, lam, x, fields, tab);
}

int deps_form_run(const mbem_op *dop, const double2 *x, const double2 *lam, double2 *out, hipStream_t s) {
    const mbem_mesh *m = dop->mesh;
    const int64_t nq = m->nt * kQP, tiles = (nq + kShapeTile - 1) / kShapeTile;
    const bool nodal = dop->p.frame == MBEM_FRAME_NODAL;
    if (tiles > 65535 || 3 * m->n_spairs > 0x7fffffffLL) { set_error("too many pairs for one launch"); return MBEM_EINVAL; }
    double2 *tab = nullptr;
    if (dev_malloc((void **)&tab, sizeof(double2) * (kTab * nq + kFormSlots + 8 * nq)) != hipSuccess) {
        set_error("permittivity gradient workspace: out of memory");
        return MBEM_ENOMEM;
    }
    double2 *slots = tab + kTab * nq;
    double *fields = (double *)(slots + kFormSlots);
    (void)hipMemsetAsync(slots, 0, sizeof(double2) * kFormSlots, s);
    launch_fields(dop, x, lam, fields, tab, s);
    hipLaunchKernelGGL(k_deps_regular, dim3((unsigned)tiles, (unsigned)tiles), dim3(kShapeTile), 0, s, nq, tab, m->d_qp,
                       fields, m->d_tri, shape_const(dop), cxd{dop->ce.x, dop->ce.y}, cxd{dop->cm.x, dop->cm.y},
                       dop->d_kconst, slots);
    int st = MBEM_OK;
    double *points = nullptr;
    if (m->n_spairs > 0) {
        ShapeSsqArgs a = ssq_args(dop, x, lam);
        st = ssq_table(a.order, &points, &a.np, s);
        a.tab = points;
        auto k = nodal ? k_deps_ssq<true> : k_deps_ssq<false>;
        if (st == MBEM_OK) hipLaunchKernelGGL(k, dim3((unsigned)(3 * a.npairs)), dim3(64), 0, s, a, slots);
    }
    hipLaunchKernelGGL(k_form_sum, dim3(1), dim3(64), 0, s, slots, out);
    const hipError_t e = hipGetLastError();
    if (st == MBEM_OK && e != hipSuccess) {
        set_error(std::string("permittivity gradient launch: ") + hipGetErrorString(e));
        st = MBEM_EDEVICE;
    }
    // their next user's work follows on the same stream
    if (points) (void)dev_free(points);
    (void)dev_free(tab);
    return st;
}

int shape_grad_run(const mbem_op *op, const mbem_params *p, const double2 *x, const double2 *lam,
                   const double *khat, const double2 *pol, const double *dir, double *dnode, double *dx,
                   hipStream_t s) {
    const mbem_mesh *m = op->mesh;
    const int64_t nt = m->nt, nq = nt * kQP, nn = m->nn;
    double *fields = nullptr, *acc = nullptr, *qb = nullptr, *nodeb = nullptr, *nodeb_x = nullptr;
    double2 *tab = nullptr;
    auto cleanup = [&]() {
        if (fields) (void)dev_free(fields);
        if (acc) (void)dev_free(acc);
        if (tab) (void)dev_free(tab);
        if (qb) (void)dev_free(qb);
        if (nodeb) (void)dev_free(nodeb);
        if (nodeb_x) (void)dev_free(nodeb_x);
    };
    const bool nodal = op->p.frame == MBEM_FRAME_NODAL;
    const int kS = nodal ? kQBN : kQB;
    if (dev_malloc((void **)&fields, sizeof(double) * 16 * nq) != hipSuccess ||
        dev_malloc((void **)&acc, sizeof(double) * 2 * kSide * nq) != hipSuccess ||
        dev_malloc((void **)&tab, sizeof(double2) * kTab * nq) != hipSuccess ||
        dev_malloc((void **)&qb, sizeof(double) * kS * nq) != hipSuccess ||
        dev_malloc((void **)&nodeb, sizeof(double) * 9 * nn) != hipSuccess ||
        dev_malloc((void **)&nodeb_x, sizeof(double) * 9 * nn) != hipSuccess) {
        cleanup();
        set_error("shape gradient workspace: out of memory");
        return MBEM_ENOMEM;
    }
    int st = MBEM_OK;
    auto launch_ok = [&]() {
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) { set_error(std::string("shape gradient launch: ") + hipGetErrorString(e)); st = MBEM_EDEVICE; }
        return st == MBEM_OK;
    };
    (void)hipMemsetAsync(acc, 0, sizeof(double) * 2 * kSide * nq, s);
    (void)hipMemsetAsync(nodeb, 0, sizeof(double) * 9 * nn, s);
    (void)hipMemsetAsync(nodeb_x, 0, sizeof(double) * 9 * nn, s);
    const unsigned gq = (unsigned)((nq + 255) / 256);
    const ShapeConst C = shape_const(op);
    launch_fields(op, x, lam, fields, tab, s);
    if (launch_ok()) {
        // a small mesh divides the 64 steps over up to four wavefronts
        const int64_t tiles = (nq + kShapeTile - 1) / kShapeTile;
        const int parts = tiles * tiles >= 2048 ? 1 : tiles * tiles >= 1024 ? 2 : 4;
        hipLaunchKernelGGL(k_shape_regular, dim3((unsigned)(tiles * parts), (unsigned)tiles), dim3(kShapeTile), 0, s,
                           nq, (int)tiles, kShapeTile / parts, tab, m->d_tri, C, op->d_kconst, acc);
        launch_ok();
    }
    if (st == MBEM_OK) {
        SingleArgs sa;
        sa.khat = {khat[0], khat[1], khat[2]};
        for (int c = 0; c < 3; ++c) { sa.pol[c] = {pol[c].x, pol[c].y}; sa.ec[c] = {pol[c].x, -pol[c].y}; }
        sa.ka = p->k0;
        sa.ce = {op->ce.x, op->ce.y};
        sa.cm = {op->cm.x, op->cm.y};
        if (nodal) hipLaunchKernelGGL(k_shape_single<true>, dim3(gq), dim3(256), 0, s, nt, m->d_qp, fields, sa, acc, qb);
        else hipLaunchKernelGGL(k_shape_single<false>, dim3(gq), dim3(256), 0, s, nt, m->d_qp, fields, sa, acc, qb);
        launch_ok();
    }
    if (st == MBEM_OK) {
        if (nodal)
            hipLaunchKernelGGL(k_qp_backprop<true>, dim3(gq), dim3(256), 0, s, nt, op->n2, m->d_xyz, m->d_frames,
                               m->d_tri, lam, x, qb, nodeb);
        else
            hipLaunchKernelGGL(k_qp_backprop<false>, dim3(gq), dim3(256), 0, s, nt, op->n2, m->d_xyz, m->d_frames,
                               m->d_tri, lam, x, qb, nodeb);
        launch_ok();
    }
    if (st == MBEM_OK && m->n_spairs > 0) {
        ShapeSsqArgs a = ssq_args(op, x, lam);
        a.nodeb = nodeb;
        double *points = nullptr;
        st = ssq_table(a.order, &points, &a.np, s);
        if (st == MBEM_OK && 3 * a.npairs > 0x7fffffffLL) { set_error("too many singular pairs for one launch"); st = MBEM_EINVAL; }
        if (st == MBEM_OK) {
            a.tab = points;
            const dim3 grid((unsigned)(3 * a.npairs));
            if (nodal) hipLaunchKernelGGL(k_shape_ssq<true>, grid, dim3(64), 0, s, a);
            else hipLaunchKernelGGL(k_shape_ssq<false>, grid, dim3(64), 0, s, a);
            launch_ok();
        }
        if (points) (void)dev_free(points);            // its next user's work follows on the same stream
    }
    if (st == MBEM_OK) {
        // position adjoints so far, then the frame path adds to the copy
        (void)hipMemcpyAsync(nodeb_x, nodeb, sizeof(double) * 9 * nn, hipMemcpyDeviceToDevice, s);
        hipLaunchKernelGGL(k_frames_backprop, dim3((unsigned)((nn + 255) / 256)), dim3(256), 0, s, nn, m->d_xyz,
                           m->d_tri, m->d_inc_ptr, m->d_inc, (const double *)nodeb, nodeb_x);
        launch_ok();
    }
    if (st == MBEM_OK) {
        hipLaunchKernelGGL(k_shape_out, dim3((unsigned)((nn + 255) / 256)), dim3(256), 0, s, nn,
                           4.0 * 3.14159265358979323846 / p->k0, m->d_frames, dir, (const double *)nodeb_x, dnode,
                           dx);
        launch_ok();
    }
    if (hipStreamSynchronize(s) != hipSuccess && st == MBEM_OK) { set_error("shape gradient failed"); st = MBEM_EDEVICE; }
    cleanup();
    return st;
}

}  // namespace mbem
