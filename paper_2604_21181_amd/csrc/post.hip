// Excitation and post-processing: plane-wave right-hand sides (eqs. rhs_E,
// rhs_H), far field of the equivalent currents and the absorbed power.
#include "mbem_internal.h"
#include "p2_device.h"

namespace mbem {

constexpr int kW2 = 64;

__device__ inline double wsum(double v) {
#pragma unroll
    for (int o = kW2 / 2; o > 0; o >>= 1) v += __shfl_down(v, o, kW2);
    return v;
}

__device__ inline cx<double> cexpi(double ph) {
    double s, c;
    sincos(ph, &s, &c);
    return {c, s};
}

// Basis tangent of local node kk, component bb, at point i of the 7-point
// table: the interpolated frame (frame 0) or the projected nodal tangent.
__device__ inline dvec3 basis_at(int frame, const double *__restrict__ qp, int64_t nq, int64_t i,
                                 const double *__restrict__ frames, int64_t node, int bb) {
    if (frame == 0) {
        const int c = bb ? QT2 : QT1;
        return {qp[c * nq + i], qp[(c + 1) * nq + i], qp[(c + 2) * nq + i]};
    }
    const dvec3 n = {qp[QN * nq + i], qp[(QN + 1) * nq + i], qp[(QN + 2) * nq + i]};
    return project_tangent(nodal_tangent(frames, node, bb), n);
}

// One thread per (quadrature point, right-hand side):
//   b_E[2i+a] += -eps_a W N_i s_a.E,  b_H[2i+a] += mu_a W N_i s_a.H
// with s_a the rotated test vector of node i (frame 0: of the point).
__global__ void k_rhs(int64_t nt, int64_t n2, int nrhs, const double *__restrict__ qp,
                      const int32_t *__restrict__ tri, const double *__restrict__ frames, int frame,
                      const double *__restrict__ khat, const double2 *__restrict__ pol, double ka,
                      double2 *__restrict__ b) {
    const int64_t nq = nt * kQP;
    const int64_t id = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (id >= nq * nrhs) return;
    const int64_t i = id % nq;
    const int r = (int)(id / nq);
    const int64_t e = i / kQP;
    const int q = (int)(i % kQP);
    const dvec3 x = {qp[QX * nq + i], qp[(QX + 1) * nq + i], qp[(QX + 2) * nq + i]};
    const dvec3 s0[2] = {{qp[QS1 * nq + i], qp[(QS1 + 1) * nq + i], qp[(QS1 + 2) * nq + i]},
                         {qp[QS2 * nq + i], qp[(QS2 + 1) * nq + i], qp[(QS2 + 2) * nq + i]}};
    const dvec3 n = {qp[QN * nq + i], qp[(QN + 1) * nq + i], qp[(QN + 2) * nq + i]};
    const double W = qp[QW * nq + i];
    const dvec3 k = {khat[3 * r], khat[3 * r + 1], khat[3 * r + 2]};
    const cx<double> ph = cexpi(ka * dot(k, x));
    const cx<double> E[3] = {ph * cx<double>{pol[3 * r].x, pol[3 * r].y},
                             ph * cx<double>{pol[3 * r + 1].x, pol[3 * r + 1].y},
                             ph * cx<double>{pol[3 * r + 2].x, pol[3 * r + 2].y}};
    // H = khat x E
    const cx<double> H[3] = {k.y * E[2] - k.z * E[1], k.z * E[0] - k.x * E[2], k.x * E[1] - k.y * E[0]};
    double xi, eta, w, N[6], d1[6], d2[6];
    rule7(q, xi, eta, w);
    p2_shape(xi, eta, N, d1, d2);
    double2 *bc = b + (int64_t)r * 2 * n2;
    for (int a = 0; a < 2; ++a) {
        for (int kk = 0; kk < 6; ++kk) {
            const int64_t node = tri[6 * e + kk];
            const dvec3 s = frame == 0 ? s0[a] : cross(nodal_tangent(frames, node, a), n);
            const cx<double> sE = s.x * E[0] + s.y * E[1] + s.z * E[2];
            const cx<double> sH = s.x * H[0] + s.y * H[1] + s.z * H[2];
            const int64_t row = 2 * node + a;
            const double f = W * N[kk];
            unsafeAtomicAdd(&bc[row].x, -f * sE.re);
            unsafeAtomicAdd(&bc[row].y, -f * sE.im);
            unsafeAtomicAdd(&bc[n2 + row].x, f * sH.re);
            unsafeAtomicAdd(&bc[n2 + row].y, f * sH.im);
        }
    }
}

int rhs_run(const mbem_mesh *m, const mbem_params *p, const double *khat, const double2 *pol,
            int nrhs, double2 *b, hipStream_t s) {
    const int64_t n2 = 2 * m->nn;
    MBEM_HIP(hipMemsetAsync(b, 0, sizeof(double2) * 2 * n2 * nrhs, s));
    const int64_t n = m->nt * kQP * nrhs;
    hipLaunchKernelGGL(k_rhs, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, m->nt, n2, nrhs,
                       m->d_qp, m->d_tri, m->d_frames, p->frame, khat, pol, p->k0, b);
    MBEM_HIP(hipGetLastError());
    return MBEM_OK;
}

// Surface currents W j, W j_m at every quadrature point for g solutions
// (blockIdx.y): cur[i][12 v ..] = W j (3 complex) and W j_m of solution v, and
// the points' coordinates pos[3][np].  Points nq .. np - 1 are zeros.
__global__ __launch_bounds__(64) void k_currents(int64_t nt, int64_t n2, const double *__restrict__ qp,
                           const int32_t *__restrict__ tri, const double *__restrict__ frames, int frame,
                           const double2 *__restrict__ x, int g, int64_t np, double *__restrict__ pos,
                           double *__restrict__ cur) {
    const int64_t nq = nt * kQP;
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= np) return;
    double *o = cur + 12 * (i * g + blockIdx.y);
    if (blockIdx.y == 0)
        for (int d = 0; d < 3; ++d) pos[d * np + i] = i < nq ? qp[(QX + d) * nq + i] : 0.0;
    if (i >= nq) {
        for (int d = 0; d < 12; ++d) o[d] = 0.0;
        return;
    }
    x += (int64_t)blockIdx.y * 2 * n2;
    const int64_t e = i / kQP;
    const int q = (int)(i % kQP);
    const double W = qp[QW * nq + i];
    double xi, eta, w, N[6], d1[6], d2[6];
    rule7(q, xi, eta, w);
    p2_shape(xi, eta, N, d1, d2);
    cx<double> J[3] = {{0, 0}, {0, 0}, {0, 0}}, Jm[3] = {{0, 0}, {0, 0}, {0, 0}};
    for (int kk = 0; kk < 6; ++kk) {
        const int64_t node = tri[6 * e + kk];
        for (int bb = 0; bb < 2; ++bb) {
            const double2 cj = x[2 * node + bb], cm = x[n2 + 2 * node + bb];
            const dvec3 t = basis_at(frame, qp, nq, i, frames, node, bb);
            const double c[3] = {t.x, t.y, t.z};
            for (int d = 0; d < 3; ++d) {
                const double f = W * N[kk] * c[d];
                J[d] = J[d] + cx<double>{f * cj.x, f * cj.y};
                Jm[d] = Jm[d] + cx<double>{f * cm.x, f * cm.y};
            }
        }
    }
    for (int d = 0; d < 3; ++d) {
        o[2 * d] = J[d].re; o[2 * d + 1] = J[d].im;
        o[6 + 2 * d] = Jm[d].re; o[6 + 2 * d + 1] = Jm[d].im;
    }
}

// F(r) = (i k / 4 pi) r x sum_q e^{-i k r.y_q} (W j x r - W j_m)
//      = (i k / 4 pi) r x (A x r - B),  [A B] = sum_q e^{-i k r.y_q} W [j j_m]:
// a product of the phases (directions by points) and the currents (points by
// 12 reals per solution) on the FP64 matrix cores, the phases evaluated in the
// registers that the instruction reads.  A wavefront takes 16 directions and
// one run of points (a multiple of 4) for up to four solutions; lane l is
// direction l % 16, point l / 16 and column l % 16 of each of NT tiles of
// columns.  Cosine and sine multiply the same currents, so the complex product
// is one exchange of neighbouring columns at the end.
// Bound by the matrix units for four solutions (6 instructions per 4 points)
// and by the sine and cosine for one.  2592 directions, us, a workgroup per
// direction and solution -> this:
//   1280 triangles  one solution 259 -> 112   four  829 -> 173
//   5120 triangles  one          936 -> 327   four 3194 -> 549
// and 4 solutions, 100 directions, 1280 triangles 191 -> 56.  The wavefronts per
// SIMD (__launch_bounds__) keep the sums out of the accumulation registers,
// whose copies in every turn cost 255 us in place of 198.
typedef double f64x4p __attribute__((ext_vector_type(4)));
constexpr int kFarDirs = 16;                  // directions of a wavefront
constexpr int kFarGroup = 4;                  // solutions of a launch
constexpr int64_t kFarSlab = 32768;           // directions of a launch

template <int NT>
__global__ __launch_bounds__(256, 2) void k_farfield(int64_t np, const double *__restrict__ pos,
                                                     const double *__restrict__ cur, int nc,
                                                     const double *__restrict__ rhat, int64_t ndir, double ka,
                                                     int tiles, int run, double *__restrict__ part) {
    const int64_t wave = blockIdx.x * (int64_t)4 + __builtin_amdgcn_readfirstlane(threadIdx.x / kW2);
    const int lane = threadIdx.x % kW2, grp = lane / 16, l16 = lane % 16;
    const int64_t tile = wave % tiles, split = wave / tiles, p0 = split * run;
    if (p0 >= np) return;
    const int n = (int)(p0 + run < np ? run : np - p0);       // a multiple of 4
    const int64_t d = tile * kFarDirs + l16 < ndir ? tile * kFarDirs + l16 : ndir - 1;
    const dvec3 r = {rhat[3 * d], rhat[3 * d + 1], rhat[3 * d + 2]};
    const double *px = pos + p0, *py = px + np, *pz = py + np, *pc = cur + p0 * nc;
    uint32_t col[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) col[t] = grp * nc + (16 * t + l16 < nc ? 16 * t + l16 : 0);
    f64x4p ac[NT], as[NT];
    // returns whether a phase is beyond the short reduction's range
    auto sums = [&](auto exact) {
        bool far = false;
#pragma unroll
        for (int t = 0; t < NT; ++t) ac[t] = as[t] = f64x4p{0.0, 0.0, 0.0, 0.0};
        struct Points { double x, y, z, b[NT]; };
        auto load = [&](int p) {                       // 4 points; p < n + 4
            Points v;
            v.x = px[(uint32_t)(p + grp)];
            v.y = py[(uint32_t)(p + grp)];
            v.z = pz[(uint32_t)(p + grp)];
#pragma unroll
            for (int t = 0; t < NT; ++t) v.b[t] = pc[(uint32_t)(p * nc) + col[t]];
            return v;
        };
        auto add = [&](const Points &v) {
            const double ph = -ka * dot(r, dvec3{v.x, v.y, v.z});
            double sn, cs;
            if constexpr (decltype(exact)::value) {
                sincos(ph, &sn, &cs);
            } else {
                far |= !(fabs(ph) < 1048576.0);
                sincos_t(ph, &sn, &cs);
            }
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                ac[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(cs, v.b[t], ac[t], 0, 0, 0);
                as[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(sn, v.b[t], as[t], 0, 0, 0);
            }
        };
        Points a = load(0);                            // the next points are loaded ahead of these
        int p = 0;
        for (; p + 8 <= n; p += 8) {
            const Points b = load(p + 4);
            add(a);
            a = load(p + 8);
            add(b);
        }
        if (p < n) add(a);
        return far;
    };
    if (__any(sums(std::false_type{}))) sums(std::true_type{});
    // (lane, e): direction grp + 4 e, column l16; even columns are real parts
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const double o = __shfl_xor(as[t][e], 1, kW2);
            const double v = ac[t][e] + (l16 & 1 ? o : -o);
            const int64_t dir = tile * kFarDirs + grp + 4 * e;
            if (dir < ndir && 16 * t + l16 < nc) part[(split * ndir + dir) * nc + 16 * t + l16] = v;
        }
}

// sums the runs and applies F = (i k / 4 pi) r x (A x r - B): one thread per
// (direction, solution, component of A or B), 16 of the first two a workgroup
__global__ __launch_bounds__(192) void k_farfield_sum(const double *__restrict__ part, int64_t ndir, int g,
                                                      int splits, const double *__restrict__ rhat, double ka,
                                                      int64_t stride, double2 *__restrict__ F) {
    __shared__ double s[16][12];
    const int64_t n = ndir * g, item = blockIdx.x * (int64_t)16 + threadIdx.x / 12;
    const int c = threadIdx.x % 12;
    double a = 0.0;
    if (item < n) {
#pragma unroll 8
        for (int k = 0; k < splits; ++k) a += part[(k * n + item) * 12 + c];
    }
    s[threadIdx.x / 12][c] = a;
    __syncthreads();
    const int64_t it = blockIdx.x * (int64_t)16 + threadIdx.x;
    if (threadIdx.x >= 16 || it >= n) return;
    const double *q = s[threadIdx.x];
    const int64_t d = it / g, v = it % g;
    const dvec3 r = {rhat[3 * d], rhat[3 * d + 1], rhat[3 * d + 2]};
    const cx<double> A[3] = {{q[0], q[1]}, {q[2], q[3]}, {q[4], q[5]}};
    const cx<double> B[3] = {{q[6], q[7]}, {q[8], q[9]}, {q[10], q[11]}};
    const cx<double> w[3] = {r.z * A[1] - r.y * A[2] - B[0], r.x * A[2] - r.z * A[0] - B[1],
                             r.y * A[0] - r.x * A[1] - B[2]};
    const cx<double> o[3] = {r.y * w[2] - r.z * w[1], r.z * w[0] - r.x * w[2], r.x * w[1] - r.y * w[0]};
    const double f = ka * 0.079577471545947667884;
    for (int k = 0; k < 3; ++k) F[v * stride + 3 * d + k] = {-f * o[k].im, f * o[k].re};
}

// Points of a run (a multiple of 4): enough wavefronts for four a SIMD, at most
// 64 runs, since the sum over them is a serial chain, none below 64 points, and
// none so long that a 32-bit offset would not reach its end.
static int64_t far_run(int64_t np, int64_t tiles) {
    const int64_t want = std::max<int64_t>(std::min<int64_t>({(4096 + tiles - 1) / tiles, 64, (np + 63) / 64}),
                                           (np >> 20) + 1);
    const int64_t run = (np + want - 1) / want;
    return (run + 3) / 4 * 4;
}

int farfield_run(const mbem_mesh *m, const mbem_params *p, const double2 *x, int nrhs,
                 const double *rhat, int64_t ndir, double2 *F, hipStream_t s) {
    const int64_t nq = m->nt * kQP, np = (nq + 3) / 4 * 4, n2 = 2 * m->nn, stride = 3 * ndir;
    if (ndir <= 0) return MBEM_OK;
    const int gmax = std::min(nrhs, kFarGroup);
    int64_t room = 0;
    for (int64_t d0 = 0; d0 < ndir; d0 += kFarSlab) {
        const int64_t nd = std::min(kFarSlab, ndir - d0), run = far_run(np, (nd + kFarDirs - 1) / kFarDirs);
        room = std::max(room, (np + run - 1) / run * nd);
    }
    // the partial sums behind the points: the loads ahead of the last points of
    // pos and cur (4 points at most) stay inside
    double *pos = nullptr;
    MBEM_HIP(dev_malloc((void **)&pos, sizeof(double) * (3 * np + 12 * (np + 4 + room) * gmax)));
    double *cur = pos + 3 * np, *part = cur + 12 * (np + 4) * gmax;
    for (int v = 0; v < nrhs; v += kFarGroup) {
        const int g = std::min(kFarGroup, nrhs - v), nc = 12 * g;
        hipLaunchKernelGGL(k_currents, dim3((unsigned)((np + 63) / 64), g), dim3(64), 0, s, m->nt, n2,
                           m->d_qp, m->d_tri, m->d_frames, p->frame, x + (int64_t)v * 2 * n2, g, np, pos, cur);
        for (int64_t d0 = 0; d0 < ndir; d0 += kFarSlab) {
            const int64_t nd = std::min(kFarSlab, ndir - d0), tiles = (nd + kFarDirs - 1) / kFarDirs;
            const int64_t run = far_run(np, tiles), splits = (np + run - 1) / run;
            auto k = g == 1 ? k_farfield<1> : g == 2 ? k_farfield<2> : k_farfield<3>;
            hipLaunchKernelGGL(k, dim3((unsigned)((tiles * splits + 3) / 4)), dim3(256), 0, s, np, pos, cur, nc,
                               rhat + 3 * d0, nd, p->k0, (int)tiles, (int)run, part);
            hipLaunchKernelGGL(k_farfield_sum, dim3((unsigned)((nd * g + 15) / 16)), dim3(192), 0, s, part, nd, g,
                               (int)splits, rhat + 3 * d0, p->k0, stride, F + v * stride + 3 * d0);
        }
    }
    const hipError_t e = hipGetLastError();
    MBEM_HIP(dev_free(pos));
    MBEM_HIP(e);
    return MBEM_OK;
}

// sum_q Re n.(W j_m x conj(j)) with j from the unweighted coefficients.
__global__ __launch_bounds__(256) void k_absorbed(int64_t nt, int64_t n2, const double *__restrict__ qp,
                                                  const int32_t *__restrict__ tri,
                                                  const double *__restrict__ frames, int frame,
                                                  const double2 *__restrict__ x, double *out) {
    const int64_t nq = nt * kQP;
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    double v = 0.0;
    if (i < nq) {
        const int64_t e = i / kQP;
        const int q = (int)(i % kQP);
        const dvec3 n = {qp[QN * nq + i], qp[(QN + 1) * nq + i], qp[(QN + 2) * nq + i]};
        double xi, eta, w, N[6], d1[6], d2[6];
        rule7(q, xi, eta, w);
        p2_shape(xi, eta, N, d1, d2);
        cx<double> J[3] = {{0, 0}, {0, 0}, {0, 0}}, Jm[3] = {{0, 0}, {0, 0}, {0, 0}};
        for (int kk = 0; kk < 6; ++kk) {
            const int64_t node = tri[6 * e + kk];
            for (int bb = 0; bb < 2; ++bb) {
                const double2 cj = x[2 * node + bb], cm = x[n2 + 2 * node + bb];
                const dvec3 t = basis_at(frame, qp, nq, i, frames, node, bb);
                const double c[3] = {t.x, t.y, t.z};
                for (int d = 0; d < 3; ++d) {
                    J[d] = J[d] + cx<double>{N[kk] * c[d] * cj.x, N[kk] * c[d] * cj.y};
                    Jm[d] = Jm[d] + cx<double>{N[kk] * c[d] * cm.x, N[kk] * c[d] * cm.y};
                }
            }
        }
        // j_m x conj(j)
        const cx<double> Jc[3] = {{J[0].re, -J[0].im}, {J[1].re, -J[1].im}, {J[2].re, -J[2].im}};
        const cx<double> c[3] = {Jm[1] * Jc[2] - Jm[2] * Jc[1], Jm[2] * Jc[0] - Jm[0] * Jc[2],
                                 Jm[0] * Jc[1] - Jm[1] * Jc[0]};
        v = qp[QW * nq + i] * (n.x * c[0].re + n.y * c[1].re + n.z * c[2].re);
    }
    v = wsum(v);
    if (threadIdx.x % kW2 == 0) unsafeAtomicAdd(out, v);
}

int absorbed_run(const mbem_mesh *m, const mbem_params *p, const double2 *x, double *out_dev, hipStream_t s) {
    const int64_t nq = m->nt * kQP;
    MBEM_HIP(hipMemsetAsync(out_dev, 0, sizeof(double), s));
    hipLaunchKernelGGL(k_absorbed, dim3((unsigned)((nq + 255) / 256)), dim3(256), 0, s, m->nt, 2 * m->nn,
                       m->d_qp, m->d_tri, m->d_frames, p->frame, x, out_dev);
    MBEM_HIP(hipGetLastError());
    return MBEM_OK;
}

// sum_d w_d |F_d|^2 over ndir directions (3 complex components each)
__global__ __launch_bounds__(256) void k_wnorm(int64_t ndir, const double2 *F, const double *w, double *out) {
    const int64_t d = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    double v = 0;
    if (d < ndir)
        for (int k = 0; k < 3; ++k) v += w[d] * (F[3 * d + k].x * F[3 * d + k].x + F[3 * d + k].y * F[3 * d + k].y);
    v = wsum(v);
    if (threadIdx.x % kW2 == 0) unsafeAtomicAdd(out, v);
}

int weighted_norm_run(int64_t ndir, const double2 *F, const double *w, double *out, hipStream_t s) {
    MBEM_HIP(hipMemsetAsync(out, 0, sizeof(double), s));
    hipLaunchKernelGGL(k_wnorm, dim3((unsigned)((ndir + 255) / 256)), dim3(256), 0, s, ndir, F, w, out);
    MBEM_HIP(hipGetLastError());
    return MBEM_OK;
}

}  // namespace mbem
