// Singular element pairs of the fills (Sec. 4.2, 6.1): coincident, common
// edge, common vertex, by Sauter-Schwab quadrature, 6 / 5 / 2 regions x n^4
// Gauss points, in FP64; the full kernels or their eps_i derivatives, or the
// paper's scheme (the singular kernels kappa^s there, and the remainders
// kappa - kappa^s on the 12-point rule).
//
// Every lane evaluates one quadrature point per batch (kernel values and
// shape functions) into LDS; then 24 lanes, one real component (2 c + re/im)
// of the twelve kernel values each, times kStreams streams of points add up
// the 6 x 6 products N_i(x) N_j(y) kappa in registers.  In every region one of
// the two points does not depend on the innermost variable: n consecutive
// points (a group) share it, so the sum over a group is contracted with the
// other side first and with the shared side once: 60 instead of 168
// multiply-adds per four points and component.
//
// Bound by vector arithmetic in the point evaluations (0.8 ms of the 1.1 ms
// below) and LDS reads in the products, at two wavefronts per SIMD (the 36
// sums stay live).  The points and weights are the same for all pairs of a
// class: read from a table built once per fill instead of decoded by every
// lane.  The triangles' positions and tangents are polynomials in LDS: as
// uniform node data they filled the scalar file (170 - 214 spills).  On the
// 1280-triangle sphere, with one P2 sum per node and one product per point
// before -> now: 1.51 -> 1.16 ms; node-attached tangents 3.25 -> 2.63;
// paper's scheme 1.65 -> 1.09, node-attached 3.75 -> 2.67; 80 triangles
// 177 -> 115 us (136 us with a workgroup per pair instead of per two regions).
// Blocks of a 70-, an 80- and a 320-triangle body, four media, both rules and
// bases, against an 80-bit evaluation, with one P2 sum per node -> now: K1 5.0e-16
// to 1.6e-15 -> 4.9e-16 to 1.7e-15 (12-point rule at large |k|: up to 8 % more, else
// equal or less), K2^eps 5.9e-16 to 1.9e-14 -> 4.0e-16 to 3.2e-15, K2^mu 2.9 to
// 5.9e-16 -> 2.8 to 5.1e-16.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "kappa.h"
#include "kappa64.h"
#include "mbem_internal.h"
#include "near_store.h"
#include "p2_device.h"
#include "ssq_map.h"

namespace mbem {

namespace {

__device__ inline void atomic_add(double *p, double v) { unsafeAtomicAdd(p, v); }
__device__ inline void atomic_add(float *p, double v) { unsafeAtomicAdd(p, (float)v); }

constexpr int kRuleGroup = 4;                         // remainder points per group (12 share x)

// Gauss-Legendre points and weights on [0, 1]
struct GaussRule {
    double x[kMaxSSQ], w[kMaxSSQ];
};

// Point table, fields s1, t1, s2, t2, weight (Jacobian included); a negative
// weight marks the points whose y does not depend on the innermost variable
// (else x does not).  The remainder points hold xi, eta of both triangles: as
// s, t they would come back rounded, the same way on every pair.
__global__ void k_ssq_table(int n, int64_t np, GaussRule gl, double *__restrict__ tab) {
    const int64_t id = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (id >= np) return;
    const int n4 = n * n * n * n;
    double v[5];
    if (id < (int64_t)kTableRegions * n4) {
        const int reg = (int)(id / n4);
        int g = (int)(id % n4);
        const int i3 = g % n; g /= n;
        const int i2 = g % n; g /= n;
        const int i1 = g % n, i0 = g / n;
        const int cls = reg < 6 ? 3 : reg < 11 ? 2 : 1, r = reg - table_region(cls);
        const double jac = ss_region(cls, r, gl.x[i0], gl.x[i1], gl.x[i2], gl.x[i3], v[0], v[1], v[2], v[3]);
        const int xfix = cls == 3 ? 0x29 : cls == 2 ? 0x6 : 0x1;     // regions 0 3 5 / 1 2 / 0
        v[4] = jac * gl.w[i0] * gl.w[i1] * gl.w[i2] * gl.w[i3] * ((xfix >> r) & 1 ? 1.0 : -1.0);
    } else {
        // the 12-point rule on both triangles
        const int rr = (int)(id - (int64_t)kTableRegions * n4), p = rr / kQP12, q = rr % kQP12;
        double xe, ye, we, xf, yf, wf;
        rule12(p, xe, ye, we);
        rule12(q, xf, yf, wf);
        v[0] = xe; v[1] = ye; v[2] = xf; v[3] = yf;
        v[4] = we * wf;
    }
#pragma unroll
    for (int f = 0; f < 5; ++f) tab[f * np + id] = v[f];
}

// One triangle's position (relative to an origin near the pair, so that the
// distance of two close points keeps its digits) and nodal tangents as
// polynomials c0 + c1 xi + c2 eta + c3 xi^2 + c4 xi eta + c5 eta^2: coefficient
// k of field d (x, t1, t2: 9) at co[9 k + d].
constexpr int kCo = 54;
// P2 point and frame as p2_point, normalised without divisions, in two steps:
// the tangents come after the kernel scalars, which need the registers.
__device__ __forceinline__ void ssq_position(const double *co, double xi, double eta, dvec3 &x, dvec3 &n, double &J) {
    double v[3], d1[3], d2[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const double c3 = co[27 + d], c4 = co[36 + d], c5 = co[45 + d];
        const double t = fma(c3, xi, fma(c4, eta, co[9 + d])), s = fma(c5, eta, co[18 + d]);
        v[d] = fma(xi, t, fma(eta, s, co[d]));
        d1[d] = fma(c3, xi, t);
        d2[d] = fma(c4, xi, fma(c5, eta, s));
    }
    const dvec3 c = cross(dvec3{d1[0], d1[1], d1[2]}, dvec3{d2[0], d2[1], d2[2]});
    const Root64 root = root64(dot(c, c));
    J = root.r;
    n = root.inv * c;
    x = {v[0], v[1], v[2]};
}
__device__ __forceinline__ void ssq_frame(const double *co, double xi, double eta, dvec3 n, dvec3 t[2]) {
    double v[6];
#pragma unroll
    for (int d = 0; d < 6; ++d) {
        const double tt = fma(co[30 + d], xi, fma(co[39 + d], eta, co[12 + d])), s = fma(co[48 + d], eta, co[21 + d]);
        v[d] = fma(xi, tt, fma(eta, s, co[3 + d]));
    }
    dvec3 u1 = {v[0], v[1], v[2]}, u2 = {v[3], v[4], v[5]};
    u1 = u1 - dot(n, u1) * n;
    u2 = u2 - dot(n, u2) * n;
    t[0] = root64(dot(u1, u1)).inv * u1;
    u2 = u2 - dot(t[0], u2) * t[0];
    t[1] = root64(dot(u2, u2)).inv * u2;
}
__device__ __forceinline__ void p2_values(double xi, double eta, double N[6]) {
    const double l = 1.0 - xi - eta;
    N[0] = l * (2.0 * l - 1.0);
    N[1] = xi * (2.0 * xi - 1.0);
    N[2] = eta * (2.0 * eta - 1.0);
    N[3] = 4.0 * l * xi;
    N[4] = 4.0 * xi * eta;
    N[5] = 4.0 * eta * l;
}

// Singular parts of the scalars (kappa^s, Sec. 4.1 and 4.2) times w: the
// terms of negative order in R of the expansions,
//   D0^s = (k_a^2 - k_i^2)/(4 pi R), df^s = dg^s = (k_a^2 - k_i^2)/(8 pi R),
//   G_chi^s = -(chi_a - chi_i)/(4 pi R^2).
__device__ __forceinline__ KScal<double> scalars_sing64(const PairConst &K, double rinv, double w) {
    const double r1 = w * 0.079577471545947667884 * rinv, r2 = r1 * rinv;
    const cx<double> dk2 = {K.ka2 - K.ki2_re, -K.ki2_im};
    KScal<double> o;
    o.D0 = r1 * dk2;
    o.df = (0.5 * r1) * dk2;
    o.dg = o.df;
    o.Ge = (-r2) * cx<double>{1.0 - K.eps_re, -K.eps_im};
    o.Gm = (-r2) * cx<double>{1.0 - K.mu_re, -K.mu_im};
    return o;
}

// Remainders kernel - kernel^s, times w.  Below max|k| R = 1/2 (and at R = 0):
// the expansions without their singular terms, whose coefficients the host
// shifts into Kr so that only non-negative powers of R remain (D0 by one
// power, df and dg by three, G by two; truncated after n = 6); otherwise the
// closed forms minus the singular parts.
__device__ __forceinline__ KScal<double> scalars_rem64(const PairConst &K, const KernelConst &Kr, double R,
                                                       double rinv, double w) {
    KScal<double> o;
    if (R > 0.0 && K.kmax * R >= kSeriesRho) {
        const KScal<double> c = scalars_closed64(K, R, rinv, w), s = scalars_sing64(K, rinv, w);
        o.D0 = c.D0 - s.D0;
        o.df = c.df - s.df;
        o.dg = c.dg - s.dg;
        o.Ge = c.Ge - s.Ge;
        o.Gm = c.Gm - s.Gm;
        return o;
    }
    const double f = w * 0.079577471545947667884;
    o.D0 = f * horner<double, kPaperTerms - 1>(Kr.cD, R);
    o.df = f * horner<double, kPaperTerms - 3>(Kr.cF, R);
    o.dg = f * horner<double, kPaperTerms - 3>(Kr.cG, R);
    o.Ge = f * horner<double, kPaperTerms - 2>(Kr.cE, R);
    o.Gm = f * horner<double, kPaperTerms - 2>(Kr.cM, R);
    return o;
}

}  // namespace

template <typename TS>
struct SsqArgs {
    int64_t n2, npairs;
    const int32_t *pairs;   // e, f, class, perm codes
    const int32_t *tri;
    const double *xyz, *frames;
    int order;
    int64_t np;             // table points
    const double *tab;
    const KernelConst *K;   // device: series of the kernels, paper's scheme: [1] of the remainders
    PairConst kc;
    const int32_t *row_map; // null, or node -> row node of a band buffer
    int regions;            // regions of one workgroup
    TS *Z[3];
    NearView near;          // MIXED with the near store: added there in FP64
};

// Launch shape.  One LDS row per point: 24 kernel reals and the shape
// functions of the side that changes within a group; node-attached tangents
// instead of those: per node k the 2 x 2 N_k t_a,k . t_g(point).  One row per
// group for the shared side, and which side that is.  NODAL: the 2 x 2
// contractions make the consumers the larger part: four wavefronts per
// workgroup, the first two producing, all of them consuming (ten streams).
constexpr int kSsqPoints = 128;
template <bool NODAL>
struct SsqShape {
    static constexpr int threads = NODAL ? 256 : 128;
    static constexpr int streams = NODAL ? 10 : 5;
    static constexpr int shape = NODAL ? 24 : 6;                 // shape data of one side
    static constexpr int row = 24 + shape + 1, fix = shape + 1;  // odd strides
    static constexpr int groups = 64;                            // at order 2; order 1: see below
    static constexpr int words(int a, int b) { return a > b ? a : b; }
    static constexpr int lds = words(kSsqPoints * row + groups * fix, streams * 36 * 24);
};

// Regions of one workgroup: a coincident pair has 12 batches of points at
// order 4 and a common-vertex pair 4; two regions per workgroup level them.
// Into complex64 a pair stays with one workgroup: every part's block would be
// rounded to 32 bits by an addition of its own (mixed solve of a 300-triangle
// body: x off by 8.8e-8 from the 64-bit solution in parts, 8.5e-8 whole), at no
// cost on 1280 triangles (fill and product 5.23 ms in parts, 5.22 whole).
constexpr int kSsqMaxRegions = 6, kSsqSplitRegions = 2;

template <typename TS, bool DK, bool NODAL, bool PAPER>
__global__ __launch_bounds__(SsqShape<NODAL>::threads) __attribute__((amdgpu_waves_per_eu(2, 8)))
void k_ssq(SsqArgs<TS> a) {
    using Sh = SsqShape<NODAL>;
    __shared__ double s_pt[Sh::lds];
    __shared__ double s_co[2][kCo];
    __shared__ KernelConst s_K;                   // series coefficients (PAPER: of the remainders)
    __shared__ double s_tn[NODAL ? 72 : 1];       // NODAL: tangents of both triangles' nodes [side][k][b][3]
    double *const s_fx = s_pt + kSsqPoints * Sh::row;
    const int tid = threadIdx.x;
    const int64_t pid = blockIdx.x % a.npairs;
    const int part = (int)(blockIdx.x / a.npairs);
    const int32_t e = a.pairs[4 * pid], f = a.pairs[4 * pid + 1];
    const int cls = a.pairs[4 * pid + 2], code = a.pairs[4 * pid + 3];
    const int nreg = cls == 3 ? 6 : cls == 2 ? 5 : 2;
    if (a.regions * part >= nreg) return;
    const int32_t *const te = a.tri + 6 * (int64_t)e, *const tf = a.tri + 6 * (int64_t)f;
    if constexpr (NODAL) {
        if (tid < 72) {
            const int side = tid / 36, r = tid % 36, k = r / 6, b = (r / 3) % 2, d = r % 3;
            s_tn[tid] = a.frames[9 * (int64_t)(side ? tf : te)[k] + 3 + 3 * b + d];
        }
    }
    {
        constexpr int nw = (int)(sizeof(KernelConst) / sizeof(double));
        const double *src = (const double *)(a.K + (PAPER ? 1 : 0));
        for (int i = tid; i < nw; i += Sh::threads) ((double *)&s_K)[i] = src[i];
    }
    if (tid < 2 * kCo) {
        const int side = tid / kCo, k = tid % kCo / 9, d = tid % 9;
        const int32_t *t = side ? tf : te;
        double v[6];
#pragma unroll
        for (int q = 0; q < 6; ++q)
            v[q] = d < 3 ? a.xyz[3 * (int64_t)t[q] + d] - a.xyz[3 * (int64_t)te[0] + d]
                         : a.frames[9 * (int64_t)t[q] + d];
        s_co[side][9 * k + d] = p2_coef(k, v);
    }
    __syncthreads();
    const int comp = tid % 24, stream = tid / 24;    // consumer role
    const bool consumer = tid < 24 * Sh::streams;
    double acc[36];
#pragma unroll
    for (int k = 0; k < 36; ++k) acc[k] = 0.0;

    // the points [p0, p1) of the table in groups of m
    auto points = [&](int64_t p0, int64_t p1, int m, bool rem) {
        const int per = min(kSsqPoints / m, Sh::groups) * m;      // points per batch: whole groups
        for (int64_t base = p0; base < p1; base += per) {
            const int cnt = (int)min((int64_t)per, p1 - base);
            if (tid < cnt) {
                double *pt = s_pt + tid * Sh::row;
                const double *q = a.tab + base + tid;
                const double w0 = q[4 * a.np];
                const bool xfix = w0 > 0.0;
                double xe, ye, xf, yf;
                if (PAPER && rem) {
                    xe = q[0], ye = q[a.np], xf = q[2 * a.np], yf = q[3 * a.np];
                } else {
                    ss_local(code & 63, q[0], q[a.np], xe, ye);
                    ss_local(code >> 6, q[2 * a.np], q[3 * a.np], xf, yf);
                }
                dvec3 x, nx, y, ny;
                double Jx, Jy;
                ssq_position(s_co[0], xe, ye, x, nx, Jx);
                ssq_position(s_co[1], xf, yf, y, ny, Jy);
                const dvec3 Rv = x - y;
                const double d2 = dot(Rv, Rv);
                // R = 0 (remainders on a coincident pair): no direction
                const Root64 root = PAPER && d2 == 0.0 ? Root64{0.0, 0.0} : root64(d2);
                const double rinv = root.inv, R = root.r;
                const double w = fabs(w0) * Jx * Jy;
                const dvec3 Rh = rinv * Rv;
                KScal<double> sc;
                double ww = w;
                if constexpr (PAPER) {
                    sc = rem ? scalars_rem64(a.kc, s_K, R, rinv, w) : scalars_sing64(a.kc, rinv, w);
                    ww = 1.0;
                } else if constexpr (DK) {
                    sc = kernel_scalars_deps(s_K, R, rinv);
                } else if (a.kc.kmax * R < kSeriesRho) {
                    sc = kernel_scalars_series<double>(s_K, R);
                } else {
                    sc = scalars_closed64(a.kc, R, rinv, w);
                    ww = 1.0;
                }
                dvec3 ta[2], tb[2];
                ssq_frame(s_co[0], xe, ye, nx, ta);
                ssq_frame(s_co[1], xf, yf, ny, tb);
                const dvec3 sa[2] = {cross(ta[0], nx), cross(ta[1], nx)};
                cx<double> k[12];
                kappa_combine<double>(sc, Rh, nx, ta, sa, tb, ww, k);
#pragma unroll
                for (int c = 0; c < 12; ++c) { pt[2 * c] = k[c].re; pt[2 * c + 1] = k[c].im; }
                const bool head = tid % m == 0;
                double *fx = s_fx + (tid / m) * Sh::fix;
                if (head) fx[Sh::shape] = w0;
                double Nx[6], Ny[6];
                p2_values(xe, ye, Nx);
                p2_values(xf, yf, Ny);
                if constexpr (!NODAL) {
#pragma unroll
                    for (int j = 0; j < 6; ++j) {
                        pt[24 + j] = xfix ? Ny[j] : Nx[j];
                        if (head) fx[j] = xfix ? Nx[j] : Ny[j];
                    }
                } else {
                    double *px = xfix ? fx : pt + 24, *py = xfix ? pt + 24 : fx;
#pragma unroll
                    for (int j = 0; j < 6; ++j)
#pragma unroll
                        for (int b = 0; b < 2; ++b) {
                            const double *ue = s_tn + 6 * j + 3 * b, *uf = s_tn + 36 + 6 * j + 3 * b;
                            const dvec3 ve = {ue[0], ue[1], ue[2]}, vf = {uf[0], uf[1], uf[2]};
#pragma unroll
                            for (int g = 0; g < 2; ++g) {
                                if (!xfix || head) px[4 * j + 2 * b + g] = Nx[j] * dot(ve, ta[g]);
                                if (xfix || head) py[4 * j + 2 * b + g] = Ny[j] * dot(vf, tb[g]);
                            }
                        }
                }
            }
            __syncthreads();
            if (consumer) {
                const int ng = cnt / m;                           // p1 - p0 is a whole number of groups
                for (int gr = stream; gr < ng; gr += Sh::streams) {
                    const double *fx = s_fx + gr * Sh::fix, *row = s_pt + gr * m * Sh::row;
                    const bool xfix = fx[Sh::shape] > 0.0;
                    if constexpr (!NODAL) {
                        double u[6] = {0, 0, 0, 0, 0, 0};
                        for (int k = 0; k < m; ++k, row += Sh::row) {
                            const double kv = row[comp];
#pragma unroll
                            for (int j = 0; j < 6; ++j) u[j] += row[24 + j] * kv;
                        }
                        if (xfix) {
#pragma unroll
                            for (int i = 0; i < 6; ++i)
#pragma unroll
                                for (int j = 0; j < 6; ++j) acc[6 * i + j] += fx[i] * u[j];
                        } else {
#pragma unroll
                            for (int i = 0; i < 6; ++i)
#pragma unroll
                                for (int j = 0; j < 6; ++j) acc[6 * i + j] += u[i] * fx[j];
                        }
                    } else {
                        // component (c = 4 op + 2 alpha + beta, re / im): acc[i][j] +=
                        // sum_{g,d} A_i[alpha][g] B_j[beta][d] k[op, g, d]
                        const int c = comp >> 1, ri = comp & 1, al = (c >> 1) & 1, be = c & 1;
                        const int k0 = 8 * (c >> 2) + ri;         // + 4 g + 2 d
                        double u0[6] = {0, 0, 0, 0, 0, 0}, u1[6] = {0, 0, 0, 0, 0, 0};
                        if (xfix) {
                            for (int k = 0; k < m; ++k, row += Sh::row) {
                                const double k00 = row[k0], k01 = row[k0 + 2], k10 = row[k0 + 4], k11 = row[k0 + 6];
#pragma unroll
                                for (int j = 0; j < 6; ++j) {
                                    const double b0 = row[24 + 4 * j + 2 * be], b1 = row[24 + 4 * j + 2 * be + 1];
                                    u0[j] += b0 * k00 + b1 * k01;
                                    u1[j] += b0 * k10 + b1 * k11;
                                }
                            }
#pragma unroll
                            for (int i = 0; i < 6; ++i) {
                                const double a0 = fx[4 * i + 2 * al], a1 = fx[4 * i + 2 * al + 1];
#pragma unroll
                                for (int j = 0; j < 6; ++j) acc[6 * i + j] += a0 * u0[j] + a1 * u1[j];
                            }
                        } else {
                            for (int k = 0; k < m; ++k, row += Sh::row) {
                                const double k00 = row[k0], k01 = row[k0 + 2], k10 = row[k0 + 4], k11 = row[k0 + 6];
#pragma unroll
                                for (int i = 0; i < 6; ++i) {
                                    const double a0 = row[24 + 4 * i + 2 * al], a1 = row[24 + 4 * i + 2 * al + 1];
                                    u0[i] += a0 * k00 + a1 * k10;
                                    u1[i] += a0 * k01 + a1 * k11;
                                }
                            }
#pragma unroll
                            for (int j = 0; j < 6; ++j) {
                                const double b0 = fx[4 * j + 2 * be], b1 = fx[4 * j + 2 * be + 1];
#pragma unroll
                                for (int i = 0; i < 6; ++i) acc[6 * i + j] += u0[i] * b0 + u1[i] * b1;
                            }
                        }
                    }
                }
            }
            __syncthreads();
        }
    };
    const int64_t n4 = (int64_t)a.order * a.order * a.order * a.order;
    const int64_t r0 = table_region(cls);
    points((r0 + a.regions * part) * n4, (r0 + min(a.regions * (part + 1), nreg)) * n4, a.order, false);
    if constexpr (PAPER)
        if (part == 0)
            points(kTableRegions * n4, kTableRegions * n4 + kQP12 * kQP12, kRuleGroup, true);

    // the streams in a fixed order, then the workgroup's 6 x 6 x 12 block
    // (atomics: a node pair collects several element pairs and parts)
    if (consumer) {
#pragma unroll
        for (int k = 0; k < 36; ++k) s_pt[(stream * 36 + k) * 24 + comp] = acc[k];
    }
    __syncthreads();
    for (int it = tid; it < 36 * 12; it += Sh::threads) {
        const int k = it / 12, cc = it % 12;
        double re = 0, im = 0;
#pragma unroll
        for (int s = 0; s < Sh::streams; ++s) {
            re += s_pt[(s * 36 + k) * 24 + 2 * cc];
            im += s_pt[(s * 36 + k) * 24 + 2 * cc + 1];
        }
        const int i = k / 6, j = k % 6;
        const int op = cc / 4, al = (cc / 2) % 2, be = cc % 2;
        if (a.near.bits) {
            // every node pair of a singular element pair is in the pattern
            double *dst = (double *)(a.near.val + 12 * near_slot(a.near, te[i], tf[j]) + cc);
            atomic_add(dst, re);
            atomic_add(dst + 1, im);
            continue;
        }
        const int64_t tn = a.row_map ? a.row_map[te[i]] : te[i];
        const int64_t row = 2 * tn + al, col = 2 * (int64_t)tf[j] + be;
        TS *dst = (op == 0 ? a.Z[0] : op == 1 ? a.Z[1] : a.Z[2]) + 2 * (row * a.n2 + col);
        atomic_add(dst, re);
        atomic_add(dst + 1, im);
    }
}

template <typename TS>
static int launch(const mbem_op *op, bool deriv, SsqArgs<TS> &a, hipStream_t s) {
    const bool paper = op->p.quadrature == MBEM_QUAD_PAPER, nodal = op->p.frame == MBEM_FRAME_NODAL;
    // FP64 destinations: the blocks of Z, or the near store's values
    a.regions = std::is_same<TS, double>::value || a.near.bits ? kSsqSplitRegions : kSsqMaxRegions;
    const int64_t parts = kSsqMaxRegions / a.regions;
    if (parts * a.npairs > 0x7fffffffLL) { set_error("too many singular pairs for one launch"); return MBEM_EINVAL; }
    const dim3 grid((unsigned)(parts * a.npairs)), blk(nodal ? SsqShape<true>::threads : SsqShape<false>::threads);
    if (paper) {
        if (nodal) hipLaunchKernelGGL((k_ssq<TS, false, true, true>), grid, blk, 0, s, a);
        else hipLaunchKernelGGL((k_ssq<TS, false, false, true>), grid, blk, 0, s, a);
    } else if (deriv) {
        if constexpr (std::is_same<TS, double>::value) {
            if (nodal) hipLaunchKernelGGL((k_ssq<TS, true, true, false>), grid, blk, 0, s, a);
            else hipLaunchKernelGGL((k_ssq<TS, true, false, false>), grid, blk, 0, s, a);
        }
    } else {
        if (nodal) hipLaunchKernelGGL((k_ssq<TS, false, true, false>), grid, blk, 0, s, a);
        else hipLaunchKernelGGL((k_ssq<TS, false, false, false>), grid, blk, 0, s, a);
    }
    MBEM_HIP(hipGetLastError());
    return MBEM_OK;
}

int ssq_table(int n, double **tab, int64_t *np, hipStream_t s) {
    *np = (int64_t)kTableRegions * n * n * n * n + kQP12 * kQP12;
    double x[kMaxSSQ], w[kMaxSSQ];
    gauss_legendre(n, x, w);
    GaussRule gl{};
    for (int i = 0; i < n; ++i) {
        gl.x[i] = 0.5 * (1.0 + x[n - 1 - i]);
        gl.w[i] = 0.5 * w[n - 1 - i];
    }
    const hipError_t err = dev_malloc((void **)tab, sizeof(double) * 5 * *np);
    if (err != hipSuccess) { set_error(std::string("singular-pair table: ") + hipGetErrorString(err)); return MBEM_ENOMEM; }
    hipLaunchKernelGGL(k_ssq_table, dim3((unsigned)((*np + 255) / 256)), dim3(256), 0, s, n, *np, gl, *tab);
    if (hipGetLastError() != hipSuccess) {
        (void)dev_free(*tab);
        *tab = nullptr;
        set_error("singular-pair table: launch failed");
        return MBEM_EDEVICE;
    }
    return MBEM_OK;
}

template <typename TS>
static int run(mbem_op *op, bool deriv, const FillBand *band, hipStream_t s) {
    const mbem_mesh *m = op->mesh;
    SsqArgs<TS> a{};
    a.n2 = op->n2;
    a.npairs = band ? band->n_spairs : m->n_spairs;
    if (a.npairs == 0) return MBEM_OK;
    a.pairs = band ? band->spairs : m->d_spairs;
    a.row_map = band ? band->row_map : nullptr;
    a.tri = m->d_tri;
    a.xyz = m->d_xyz;
    a.frames = m->d_frames;
    a.order = op->p.ssq_order > 0 ? op->p.ssq_order : 4;
    if (a.order > kMaxSSQ) { set_error("ssq_order above 8 is not supported"); return MBEM_EINVAL; }
    a.K = op->d_kconst + 1;
    a.kc = pair_const(op->ka, op->ki, op->eps_i, op->mu_i);
    for (int o = 0; o < 3; ++o) a.Z[o] = (TS *)(band ? band->Z[o] : op->K[o]);
    a.near = band ? NearView{} : op->near_view();
    double *tab = nullptr;
    MBEM_TRY(ssq_table(a.order, &tab, &a.np, s));
    a.tab = tab;
    const int st = launch(op, deriv, a, s);
    MBEM_HIP(dev_free(tab));         // its next user's work follows on the same stream
    return st;
}

int ssq_fill_run(mbem_op *op, bool deriv, const FillBand *band, hipStream_t s) {
    return op->prec == MBEM_FP64 || band ? run<double>(op, deriv, band, s) : run<float>(op, deriv, band, s);
}

}  // namespace mbem
