// Regular element pairs of the FP64 dense operators (Sec. 4.1-4.2): the
// 7-point or the 12-point rule, the kernels or their eps_i derivatives,
// the interpolated frame or node-attached tangents.
//
// The triangles are grouped into batches of up to kPairNB that share nodes.
// Two passes per band of test batches, through a scratch that stays resident
// in the last-level cache:
//   tiles   one workgroup per (test batch, trial batch): per test triangle the
//           twelve kernel values of every point pair, contracted with the
//           trial and the test shape functions and merged by trial node, are
//           added to T[test node of the batch][slot][op, alpha, beta], a slot
//           being a (trial batch, node) pair;
//   gather  Z[2 i + alpha][2 j + beta] = the sum of T over the band's batches
//           with node i and the batches with node j.
// A launch carries the tiles of one band and, behind them, the gather of the
// band before (two scratch buffers), which fills the tail of the tiles.
//
// Adding the tiles straight to Z (one launch per pair of colour classes,
// each entry read and written 6.2 times in 32-byte pieces) was bound by that
// traffic; here an entry of Z is written once per band that touches its row
// in full rows, and what repeats stays in the cache.  No colour classes are
// needed, so the launch count does not grow with the mesh's largest node
// valence.
//
// Measured on the 1280-triangle sphere (10 248 unknowns), regular pairs by
// colour classes -> here: 6.9 -> 3.8 ms (7 points), 22.8 -> 7.1 ms (12
// points), 9.4 -> 7.5 ms (7 points, node-attached tangents), 62.5 -> 21.9 ms
// (12 points, node-attached).  Of the 3.8 ms the tiles alone take 2.85 ms:
// LDS and the non-FP64 half of their vector instructions (FP64 units 22 %
// busy); the gather alone takes 1.6 ms, of which 0.9 are not hidden.  The
// launch moves 7.3 GB out of and 7.4 GB into the L2s.
#include "mbem_internal.h"
#include "kappa.h"
#include "kappa64.h"
#include "p2_device.h"
#include "pairs.h"

namespace mbem {

namespace {

// ------------------------------------------------------- contractions --
// 12-point counterpart of contract7: the two three-point orbits as there,
// and the six-point orbit (v0, v1, v2 on the three vertices in every order)
// through the sums of the two points that give vertex k the value v_d: 47
// multiply-adds instead of 72.
__host__ __device__ constexpr double r12_v(int d) {
    return r12_bary(6, d);   // point 6 carries v_d on vertex d
}
template <typename T>
__device__ inline void contract12o(const cx<T> v[kQP12], cx<T> out[6]) {
    constexpr double a = r12_bary(0, 1), b = r12_bary(3, 1);
    constexpr double A = 1.0 - 2.0 * a, B = 1.0 - 2.0 * b;
    constexpr double Va = a * (2.0 * a - 1.0), Vb = b * (2.0 * b - 1.0);
    constexpr double Da = A * (2.0 * A - 1.0) - Va, Db = B * (2.0 * B - 1.0) - Vb;
    constexpr double Ea = 4.0 * a * A, Eb = 4.0 * b * B;
    constexpr double Ga = 4.0 * a * a - Ea, Gb = 4.0 * b * b - Eb;
    constexpr double v0 = r12_v(0), v1 = r12_v(1), v2 = r12_v(2);
    constexpr double f0 = v0 * (2.0 * v0 - 1.0), f1 = v1 * (2.0 * v1 - 1.0), f2 = v2 * (2.0 * v2 - 1.0);
    constexpr double e0 = 4.0 * v1 * v2, e1 = 4.0 * v0 * v2, e2 = 4.0 * v0 * v1;
    const cx<T> Sa = v[0] + v[1] + v[2], Sb = v[3] + v[4] + v[5];
    const cx<T> V = (T)Va * Sa + (T)Vb * Sb, E = (T)Ea * Sa + (T)Eb * Sb;
    // the two points of the six-point orbit with v_d on vertex k (points
    // 6 .. 11 hold the vertex orders 012, 021, 102, 120, 201, 210)
    const cx<T> P[3][3] = {{v[6] + v[7], v[8] + v[10], v[9] + v[11]},
                           {v[8] + v[9], v[6] + v[11], v[7] + v[10]},
                           {v[10] + v[11], v[7] + v[9], v[6] + v[8]}};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        out[k] = V + (T)Da * v[k] + (T)Db * v[3 + k] + (T)f0 * P[k][0] + (T)f1 * P[k][1] + (T)f2 * P[k][2];
        // the mid-edge node opposite vertex k: 4, 5, 3
        out[3 + (k + 1) % 3] =
            E + (T)Ga * v[k] + (T)Gb * v[3 + k] + (T)e0 * P[k][0] + (T)e1 * P[k][1] + (T)e2 * P[k][2];
    }
}

template <int NP>
__device__ __forceinline__ void contract_points(const cx<double> v[NP], cx<double> out[6]) {
    if constexpr (NP == kQP12) contract12o(v, out);
    else contract7(v, out);
}

// shape function j at point p of the rule (for the running test-side sum)
template <int NP>
__host__ __device__ constexpr double n_at(int p, int j) {
    if constexpr (NP == kQP12) {
        const double L0 = r12_bary(p, 0), L1 = r12_bary(p, 1), L2 = r12_bary(p, 2);
        return j == 0 ? L0 * (2.0 * L0 - 1.0) : j == 1 ? L1 * (2.0 * L1 - 1.0)
             : j == 2 ? L2 * (2.0 * L2 - 1.0) : j == 3 ? 4.0 * L0 * L1
             : j == 4 ? 4.0 * L1 * L2 : 4.0 * L2 * L0;
    } else {
        return n7(p, j);
    }
}

}  // namespace

// -------------------------------------------------------------- gather --
// Row tasks of one band: {node, first slot, last slot + 1, 1 if no earlier
// band wrote the node's rows} (a node's slots follow the order of the
// batches), of which the T rows row0g .. row1g - 1 are held: all of the band's,
// or a part of them where memory was short.  One workgroup per (row task, block of nodes): the T rows of the
// node's batches are read in whole runs and summed in registers, then the
// slots of every column through LDS.  A block of a single node with more than
// kPairCols slots takes several turns.
__device__ __forceinline__ void gather_rows(const PairArgs &a, int64_t id, double2 *s_v) {
    constexpr int kItems = 12 * kPairCols, kPer = (kItems + 255) / 256;
    const int tid = threadIdx.x;
    const int4 task = a.rows[id / a.ncb];
    const int cb = (int)(id % a.ncb);
    int s0 = task.y, s1 = task.z;
    while (s0 < s1 && a.slot_row[s0] < a.row0g) ++s0;
    while (s0 < s1 && a.slot_row[s1 - 1] >= a.row1g) --s1;
    if (s0 == s1) return;                  // uniform over the workgroup
    const int32_t j0 = a.cblocks[cb], j1 = a.cblocks[cb + 1];
    const int32_t p1 = a.slot_ptr[j1];
    const int ncol = 2 * (j1 - j0);
    for (int32_t p0 = a.slot_ptr[j0]; p0 < p1; p0 += kPairCols) {
        const int32_t q1 = min(p1, p0 + kPairCols);
        const int n = 12 * (q1 - p0);
        double2 v[kPer];
#pragma unroll
        for (int k = 0; k < kPer; ++k) v[k] = double2{0.0, 0.0};
        for (int s = s0; s < s1; ++s) {
            const double2 *__restrict__ row = a.Tg + ((a.slot_row[s] - a.row0g) * a.nslots + p0) * 12;
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                const double2 w = row[min(tid + 256 * k, n - 1)];   // past the end: not used below
                v[k].x += w.x;
                v[k].y += w.y;
            }
        }
        if (p0 > a.slot_ptr[j0]) __syncthreads();
#pragma unroll
        for (int k = 0; k < kPer; ++k)
            if (tid + 256 * k < kItems) s_v[tid + 256 * k] = v[k];
        __syncthreads();
        const bool first = task.w && s0 == task.y && p0 == a.slot_ptr[j0];
        for (int it = tid; it < 6 * ncol; it += 256) {
            const int g = it / ncol, c = it % ncol;
            const int32_t j = j0 + (c >> 1);
            const int32_t u0 = max(p0, a.slot_ptr[j]), u1 = min(q1, a.slot_ptr[j + 1]);
            double2 *Z = a.Z[g >> 1] + (2 * (int64_t)task.x + (g & 1)) * a.n2 + 2 * (int64_t)j0 + c;
            double2 z = {0.0, 0.0};
            if (!first) z = *Z;
            for (int32_t u = u0; u < u1; ++u) {
                const double2 w = s_v[12 * (u - p0) + 2 * g + (c & 1)];
                z.x += w.x;
                z.y += w.y;
            }
            *Z = z;
        }
    }
}

// --------------------------------------------------------------- tiles --
// One workgroup per (test batch, trial batch): everything of the trial side
// (point data, merge offsets, T columns, contraction weights) is loaded once
// and stays in registers and LDS over the test triangles.  Per test triangle
// three barriers per pass:
//  A: one point pair per lane (NP consecutive lanes: the trial points of one
//     (triangle, test point) row): kernel values into LDS, component-major;
//  B: trial side, in place: (component, triangle, test point) -> 6 nodes;
//  C: lane (g = 2 op + alpha, slot, beta): node merge, test side, T.  A row
//     of T belongs to a test node: the first triangle of the batch with the
//     node stores, the others add (the same lane, so in program order).
// The 7-point rule takes a batch in one pass of 35 rows, the 12-point rule in
// three of 20, the test side summed over the passes in registers.
// Occupancy: 51 KB of LDS, three workgroups per compute unit (two with
// node-attached tangents, whose contraction weights take 8 - 14 KB more).
template <int NP>
struct PairShape {
    static constexpr int rows = NP == kQP12 ? 20 : 35;           // (triangle, point) rows per pass
    static constexpr int passes = kPairNB * NP / rows;
    static constexpr int lanes = rows * NP;
    static constexpr int stride = NP == kQP12 ? 241 : 257;       // = 1 mod 16: components over the banks
    static_assert(passes * rows == kPairNB * NP && lanes <= 256 && lanes <= stride, "whole passes, one pair per lane");
};

template <int NP, bool DK, bool NODAL>
__global__ __launch_bounds__(256, NODAL ? 2 : 3) void k_pair_tiles(PairArgs a) {
    using Sh = PairShape<NP>;
    constexpr bool kSeries = NP == kQP;       // the 12-point scheme takes the closed forms throughout
    constexpr int kPts = NP / Sh::passes;     // test points per pass
    constexpr int kTp = kQPF * NP, kRa = NODAL ? NP * 24 : 0;
    static_assert(kPairCols <= Sh::stride, "the gather's sums fit in s_k");
    static_assert(kTp <= 256 && kRa <= 512, "test data staged by one or two loads per lane");
    __shared__ cx<double> s_k[12 * Sh::stride];
    __shared__ double s_tp[kTp];              // the test triangle's point table, field-major
    __shared__ int32_t s_te[6];
    __shared__ KernelConst s_K;               // series coefficients (unused by the 12-point rule)
    __shared__ double s_n[Sh::passes > 1 ? NP * 6 : 1];   // test shape functions at the points
    __shared__ double s_ra[NODAL ? kRa : 1];
    __shared__ double s_rb[NODAL ? kPairNB * NP * 24 : 1];
    if (blockIdx.x >= a.n_tiles) {
        gather_rows(a, blockIdx.x - a.n_tiles, (double2 *)s_k);
        return;
    }
    const int tid = threadIdx.x;
    const int32_t *__restrict__ rec = a.rec + (blockIdx.x % a.n_batches) * kPairRec;
    const int32_t *__restrict__ test = a.rec + (a.batch0 + blockIdx.x / a.n_batches) * kPairRec;
    const int64_t nq = a.nt * NP;
    const int nb = rec[0], ns = rec[1], nte = test[0];
    if constexpr (kSeries) {
        constexpr int nw = (int)(sizeof(KernelConst) / sizeof(double));
        for (int i = tid; i < nw; i += 256) ((double *)&s_K)[i] = ((const double *)a.K)[i];
    }
    if constexpr (Sh::passes > 1)
        if (tid < NP * 6) s_n[tid] = n_at<NP>(tid / 6, tid % 6);
    if constexpr (NODAL)
        for (int i = tid; i < kPairNB * NP * 24; i += 256) {
            const int fl = i / (NP * 24);
            s_rb[i] = fl < nb ? a.rtab[(int64_t)rec[kPairTri + fl] * NP * 24 + i % (NP * 24)] : 0.0;
        }
    // the test triangle's data: loaded one triangle ahead into registers
    double tp_next = 0.0, ra_next[NODAL ? 2 : 1];
    int32_t te_next = 0;
    auto load_test = [&](int64_t e) {
        if (tid < kTp) tp_next = a.qp[(int64_t)(tid / NP) * nq + e * NP + tid % NP];
        if (tid < 6) te_next = a.tri[6 * e + tid];
        if constexpr (NODAL) {
#pragma unroll
            for (int k = 0; k < 2; ++k)
                if (tid + 256 * k < kRa) ra_next[k] = a.rtab[e * kRa + tid + 256 * k];
        }
    };
    auto store_test = [&]() {
        if (tid < kTp) s_tp[tid] = tp_next;
        if (tid < 6) s_te[tid] = te_next;
    };
    auto store_ra = [&]() {
        if constexpr (NODAL) {
#pragma unroll
            for (int k = 0; k < 2; ++k)
                if (tid + 256 * k < kRa) s_ra[tid + 256 * k] = ra_next[k];
        }
    };
    load_test(test[kPairTri]);
    // A: this lane's row (kPairNB test point + triangle; the triangle is the
    // same in every pass) and trial point
    const int row = tid / NP, ql = tid % NP, fl = row % kPairNB;
    dvec3 y = {0, 0, 0}, tb[2] = {y, y};
    double wy = 0.0;
    int32_t tf[3] = {-1, -1, -1};
    if (tid < Sh::lanes && fl < nb) {
        const int64_t f = rec[kPairTri + fl];
        const double *q = a.qp + f * NP + ql;
        y = {q[0], q[nq], q[2 * nq]};
        wy = q[QW * nq];
        tb[0] = {q[QT1 * nq], q[(QT1 + 1) * nq], q[(QT1 + 2) * nq]};
        tb[1] = {q[QT2 * nq], q[(QT2 + 1) * nq], q[(QT2 + 2) * nq]};
#pragma unroll
        for (int k = 0; k < 3; ++k) tf[k] = a.tri[6 * f + k];
    }
    // C: this lane's item, its T column and its incidences (at most one per
    // triangle of the batch, eight bits each).  The batch's nodes come by
    // falling number of incidences and the lanes take them in order, so the
    // merge loop of a wavefront runs 5 + 2 + 1 + 1 times rather than 4 x 5;
    // the wavefronts take turns at the long end from workgroup to workgroup.
    const int it_c = (tid + 64 * (blockIdx.x & 3)) & 255;
    const int sl = it_c / 12, g = it_c % 12 / 2, be = it_c & 1;
    const bool item = sl < ns;
    int ninc = 0;
    uint64_t incs = 0;
    double2 *Trow = nullptr;
    if (item) {
        const int32_t *pos = rec + kPairPos, *off = rec + kPairOff, *inc = rec + kPairInc;
        const int u0 = off[sl];
        ninc = off[sl + 1] - u0;
        for (int u = 0; u < ninc; ++u) incs |= (uint64_t)inc[u0 + u] << (8 * u);
        Trow = a.T + ((test[2] - a.row0) * a.nslots + pos[sl]) * 12 + 2 * g + be;
    }
    store_test();
    store_ra();
    __syncthreads();
    for (int t = 0; t < nte; ++t) {
        if (t + 1 < nte) load_test(test[kPairTri + t + 1]);
        // rows of T of the triangle's nodes: batch node, + 256 if this triangle
        // is the batch's first with the node.  What the rows hold is loaded
        // long before it is needed: the first triangles' lines are in L2
        const int32_t *__restrict__ loc = test + kPairLoc + 6 * t;
        int32_t tloc[6];
#pragma unroll
        for (int i = 0; i < 6; ++i) tloc[i] = __builtin_amdgcn_readfirstlane(loc[i]);
        cx<double> out[6];
        auto load_rows = [&]() {
#pragma unroll
            for (int i = 0; i < 6; ++i) {
                out[i] = {0.0, 0.0};
                if (item && tloc[i] < 256) {
                    const double2 v = Trow[12 * a.nslots * tloc[i]];
                    out[i] = {v.x, v.y};
                }
            }
        };
        constexpr bool kRunning = Sh::passes > 1 || NODAL;    // out is summed point by point
        if constexpr (kRunning) load_rows();
#pragma unroll 1
        for (int s = 0; s < Sh::passes; ++s) {
            // A
            if (tid < Sh::lanes) {
                cx<double> k[12];
                bool on = tf[0] >= 0;          // singular pairs (a shared vertex) are not ours
#pragma unroll
                for (int i = 0; i < 3; ++i)
#pragma unroll
                    for (int j = 0; j < 3; ++j) on = on && (s_te[i] != tf[j]);
                if (on) {
                    const double *tp = s_tp + s * kPts + row / kPairNB;
                    auto tv = [&](int f) { return dvec3{tp[f * NP], tp[(f + 1) * NP], tp[(f + 2) * NP]}; };
                    const dvec3 Rv = tv(QX) - y;
                    const double d2 = dot(Rv, Rv);
                    const Root64 root = root64(d2);
                    const double rinv = root.inv, R = root.r;
                    const double w = tp[QW * NP] * wy;
                    KScal<double> sc;
                    double ww = w;
                    if constexpr (DK) {
                        sc = kernel_scalars_deps(s_K, R, rinv);
                    } else if (kSeries && a.kc.kmax * R < kSeriesRho) {
                        sc = kernel_scalars_series<double>(s_K, R);
                    } else {
                        sc = scalars_closed64(a.kc, R, rinv, w);
                        ww = 1.0;
                    }
                    const dvec3 ta[2] = {tv(QT1), tv(QT2)}, sa[2] = {tv(QS1), tv(QS2)};
                    kappa_combine<double>(sc, rinv * Rv, tv(QN), ta, sa, tb, ww, k);
                } else {
#pragma unroll
                    for (int c = 0; c < 12; ++c) k[c] = cx<double>{0.0, 0.0};
                }
#pragma unroll
                for (int c = 0; c < 12; ++c) s_k[c * Sh::stride + tid] = k[c];
            }
            __syncthreads();
            if (s + 1 == Sh::passes && t + 1 < nte) store_test();   // A is done with this triangle's
            if constexpr (!kRunning) load_rows();
            // B
            if constexpr (!NODAL) {
                for (int it = tid; it < 12 * Sh::rows; it += 256) {
                    cx<double> *v = s_k + (it / Sh::rows) * Sh::stride + NP * (it % Sh::rows);
                    cx<double> kv[NP], tfv[6];
#pragma unroll
                    for (int q = 0; q < NP; ++q) kv[q] = v[q];
                    contract_points<NP>(kv, tfv);
#pragma unroll
                    for (int j = 0; j < 6; ++j) v[j] = tfv[j];
                }
            } else {
                // the components (op, gamma, delta) become (op, gamma, beta)
                for (int it = tid; it < 6 * Sh::rows; it += 256) {
                    const int rw = it % Sh::rows;
                    cx<double> *v0 = s_k + 2 * (it / Sh::rows) * Sh::stride + NP * rw, *v1 = v0 + Sh::stride;
                    const double *rb = s_rb + (rw % kPairNB) * NP * 24;
                    cx<double> k0[NP], k1[NP];
#pragma unroll
                    for (int q = 0; q < NP; ++q) { k0[q] = v0[q]; k1[q] = v1[q]; }
#pragma unroll 1
                    for (int j = 0; j < 6; ++j) {
                        cx<double> o0 = {0.0, 0.0}, o1 = {0.0, 0.0};
#pragma unroll
                        for (int q = 0; q < NP; ++q) {
                            const double *w = rb + (q * 6 + j) * 4;
                            o0 = o0 + w[0] * k0[q] + w[1] * k1[q];
                            o1 = o1 + w[2] * k0[q] + w[3] * k1[q];
                        }
                        v0[j] = o0;
                        v1[j] = o1;
                    }
                }
            }
            __syncthreads();
            // C
            if (item) {
                uint64_t left = incs;
                constexpr int kStep = NP * kPairNB;      // one test point further
                if constexpr (!NODAL) {
                    cx<double> tv[kPts];
#pragma unroll
                    for (int p = 0; p < kPts; ++p) tv[p] = {0.0, 0.0};
                    const cx<double> *comp = s_k + (2 * g + be) * Sh::stride;
                    for (int u = 0; u < ninc; ++u, left >>= 8) {
                        const cx<double> *src = comp + ((int)(left >> 3) & 31) * NP + ((int)left & 7);
#pragma unroll
                        for (int p = 0; p < kPts; ++p) tv[p] = tv[p] + src[kStep * p];
                    }
                    if constexpr (Sh::passes == 1) {
                        cx<double> sum[6];
                        contract_points<NP>(tv, sum);
#pragma unroll
                        for (int i = 0; i < 6; ++i) out[i] = out[i] + sum[i];
                    } else {
#pragma unroll
                        for (int p = 0; p < kPts; ++p)
#pragma unroll
                            for (int i = 0; i < 6; ++i) out[i] = out[i] + s_n[(s * kPts + p) * 6 + i] * tv[p];
                    }
                } else {
                    // (op, gamma, beta) for gamma = 0, 1
                    const cx<double> *comp = s_k + (4 * (g >> 1) + be) * Sh::stride;
                    const double *ra = s_ra + s * kPts * 24 + 2 * (g & 1);
#pragma unroll 1
                    for (int p = 0; p < kPts; ++p, ra += 24) {
                        cx<double> t0 = {0.0, 0.0}, t1 = {0.0, 0.0};
                        left = incs;
                        for (int u = 0; u < ninc; ++u, left >>= 8) {
                            const int at = ((int)(left >> 3) & 31) * NP + ((int)left & 7) + kStep * p;
                            t0 = t0 + comp[at];
                            t1 = t1 + comp[2 * Sh::stride + at];
                        }
#pragma unroll
                        for (int i = 0; i < 6; ++i) out[i] = out[i] + ra[4 * i] * t0 + ra[4 * i + 1] * t1;
                    }
                }
                if (s + 1 == Sh::passes) {
#pragma unroll
                    for (int i = 0; i < 6; ++i)
                        Trow[12 * a.nslots * (tloc[i] & 255)] = double2{out[i].re, out[i].im};
                }
            }
            __syncthreads();
            if constexpr (NODAL) {
                // s_ra is read by C, and by no lane before the next triangle's B is done
                if (s + 1 == Sh::passes && t + 1 < nte) store_ra();
            }
        }
    }
}

// Launches of at most `part` test batches, bands in parts of that size.
template <int NP, bool DK, bool NODAL>
static int launch_bands(const mbem_op *op, PairArgs &a, int64_t part, double2 *const buf[2], hipStream_t s) {
    const mbem_mesh *m = op->mesh;
    int64_t turn = 0, band = 0;            // launches so far, band of the gather's batches
    for (int64_t b0 = 0, g0 = -1; g0 < a.n_batches;) {
        // the tiles of the batches [b0, b1), the gather of those before, [g0, b0)
        const int64_t b1 = std::min<int64_t>({b0 + part, (b0 / m->pair_band + 1) * m->pair_band, a.n_batches});
        a.n_tiles = (b1 - b0) * a.n_batches;
        if (a.n_tiles > 0) {
            a.batch0 = b0;
            a.row0 = m->pair_row0[b0];
            a.T = buf[turn & 1];
        }
        int64_t gather = 0;
        if (g0 >= 0) {
            band = g0 / m->pair_band;
            a.rows = (const int4 *)m->d_pair_rows + m->pair_rows_off[band];
            a.row0g = m->pair_row0[g0];
            a.row1g = m->pair_row0[b0];
            a.Tg = buf[(turn - 1) & 1];
            gather = (m->pair_rows_off[band + 1] - m->pair_rows_off[band]) * a.ncb;
        }
        if (a.n_tiles + gather > 0x7fffffffLL) {
            set_error("too many element pairs for one launch");
            return MBEM_EINVAL;
        }
        hipLaunchKernelGGL((k_pair_tiles<NP, DK, NODAL>), dim3((unsigned)(a.n_tiles + gather)), dim3(256), 0, s, a);
        MBEM_HIP(hipGetLastError());
        g0 = b0;
        b0 = b1;
        ++turn;
    }
    return MBEM_OK;
}

int pair_fill_run(mbem_op *op, bool deriv, hipStream_t s) {
    const mbem_mesh *m = op->mesh;
    const bool paper = op->p.quadrature == MBEM_QUAD_PAPER, nodal = op->p.frame == MBEM_FRAME_NODAL;
    PairArgs a{};
    a.nt = m->nt;
    a.n2 = op->n2;
    a.nslots = m->pair_slots;
    a.ncb = m->pair_ncb;
    a.cblocks = m->d_pair_cb;
    a.n_batches = m->pair_batches;
    a.qp = paper ? m->d_qp12 : m->d_qp;
    a.tri = m->d_tri;
    a.rec = m->d_pair_rec;
    a.slot_ptr = m->d_pair_sptr;
    a.slot_row = m->d_pair_srow;
    a.K = op->d_kconst;
    a.kc = pair_const(op->ka, op->ki, op->eps_i, op->mu_i);
    for (int o = 0; o < 3; ++o) a.Z[o] = (double2 *)op->K[o];
    if (nodal) {
        MBEM_TRY(nodal_table_f64(op, paper, s));
        a.rtab = (const double *)op->d_rtab;
    }
    // two buffers of a band, one where a single band is all; where they do not
    // fit, bands in parts, down to one batch
    int64_t part = std::min<int64_t>(m->pair_band, a.n_batches);
    double2 *scratch = nullptr, *buf[2];
    for (;;) {
        int64_t rows = 0;                  // most T rows of a part
        for (int64_t b0 = 0, b1; b0 < a.n_batches; b0 = b1) {
            b1 = std::min<int64_t>({b0 + part, (b0 / m->pair_band + 1) * m->pair_band, a.n_batches});
            rows = std::max<int64_t>(rows, m->pair_row0[b1] - m->pair_row0[b0]);
        }
        const size_t elems = (size_t)rows * 12 * a.nslots;
        const int nbuf = part < a.n_batches ? 2 : 1;
        const hipError_t err = dev_malloc((void **)&scratch, elems * sizeof(double2) * nbuf);
        buf[0] = scratch;
        buf[1] = scratch + (nbuf - 1) * elems;
        if (err == hipSuccess) break;
        if (part == 1) { set_error(std::string("fill scratch: ") + hipGetErrorString(err)); return MBEM_ENOMEM; }
        part = (part + 1) / 2;
    }
    int st;
    if (paper) st = nodal ? launch_bands<kQP12, false, true>(op, a, part, buf, s)
                          : launch_bands<kQP12, false, false>(op, a, part, buf, s);
    else if (deriv) st = nodal ? launch_bands<kQP, true, true>(op, a, part, buf, s)
                               : launch_bands<kQP, true, false>(op, a, part, buf, s);
    else st = nodal ? launch_bands<kQP, false, true>(op, a, part, buf, s)
                    : launch_bands<kQP, false, false>(op, a, part, buf, s);
    MBEM_HIP(dev_free(scratch));     // its next user's work follows on the same stream
    return st;
}

}  // namespace mbem
