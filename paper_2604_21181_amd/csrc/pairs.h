// Regular-pair fill of the FP64 dense operators (pairs.hip): trial batches
// and launch arguments.
#pragma once

#include <algorithm>
#include <cmath>

#include "mbem_internal.h"
#include "kappa64.h"
#include "p2_device.h"

namespace mbem {

struct PairArgs {
    int64_t nt, n2;
    int64_t nslots;
    int64_t batch0, n_tiles;     // first test batch and workgroups of this launch's tiles
    int32_t n_batches;
    int32_t row0, row0g, row1g;  // first T row (test node) of the tiles' and the gather's batches, end of the latter
    const double *qp;            // [kQPF][nt * points]
    const int32_t *tri;
    const int32_t *rec;          // trial batch records, kPairRec ints each
    const double *rtab;          // node-attached: [nt][points][6][2][2] tangent components
    const KernelConst *K;        // series coefficients (device)
    PairConst kc;
    double2 *T;                  // [test node of a batch][slot][4 op + 2 alpha + beta]
    // gather of the band before
    const double2 *Tg;
    int32_t ncb;                 // blocks of nodes per row
    const int32_t *cblocks;      // their first nodes, one more than blocks
    const int4 *rows;
    const int32_t *slot_ptr;     // node -> its first slot, [nn + 1]
    const int32_t *slot_row;     // slot -> its row of T
    double2 *Z[3];
};

// P2 shape functions at the points of the 7-point rule (rule7: centroid,
// then the two three-point orbits with (6 -+ sqrt 15)/21), evaluated at
// compile time: n7(q, j) = N_j(xi_q, eta_q).  The literal is sqrt(15)
// rounded to double, so the values equal those of rule7 + p2_shape.
__host__ __device__ constexpr double n7(int q, int j) {
    const double r15 = 3.8729833462074168851792653997824;
    const double s = q == 0 ? 1.0 / 3.0 : (q <= 3 ? (6.0 - r15) / 21.0 : (6.0 + r15) / 21.0);
    const int r = q == 0 ? 0 : (q - 1) % 3;
    const double xi = q == 0 ? s : (r == 1 ? 1.0 - 2.0 * s : s);
    const double eta = q == 0 ? s : (r == 2 ? 1.0 - 2.0 * s : s);
    const double L0 = 1.0 - xi - eta, L1 = xi, L2 = eta;
    return j == 0 ? L0 * (2.0 * L0 - 1.0) : j == 1 ? L1 * (2.0 * L1 - 1.0)
         : j == 2 ? L2 * (2.0 * L2 - 1.0) : j == 3 ? 4.0 * L0 * L1
         : j == 4 ? 4.0 * L1 * L2 : 4.0 * L2 * L0;
}

// out[j] = sum_q n7(q, j) v[q] through the symmetry of the rule: the three
// points of an orbit carry the same weight pattern, so with the orbit sums
// S_a = v1 + v2 + v3, S_b = v4 + v5 + v6 every vertex function is
// N(centroid) v0 + B_a S_a + B_b S_b plus (A - B) times the value at the
// orbit point nearest that vertex, and every mid-edge function
// N(centroid) v0 + E_a S_a + E_b S_b plus (F - E) times the value at the
// orbit point nearest the opposite vertex (A, B, E, F: the shape-function
// values at the orbit points).  44 real operations instead of 84.
template <typename T>
__host__ __device__ inline void contract7(const cx<T> v[7], cx<T> out[6]) {
    constexpr double c0v = n7(0, 0), c0e = n7(0, 3);
    constexpr double Ba = n7(2, 0), Bb = n7(5, 0), Da = n7(1, 0) - Ba, Db = n7(4, 0) - Bb;
    constexpr double Ea = n7(1, 3), Eb = n7(4, 3), Ga = n7(3, 3) - Ea, Gb = n7(6, 3) - Eb;
    const cx<T> Sa = v[1] + v[2] + v[3], Sb = v[4] + v[5] + v[6];
    const cx<T> V = (T)c0v * v[0] + (T)Ba * Sa + (T)Bb * Sb;
    const cx<T> E = (T)c0e * v[0] + (T)Ea * Sa + (T)Eb * Sb;
    out[0] = V + (T)Da * v[1] + (T)Db * v[4];
    out[1] = V + (T)Da * v[2] + (T)Db * v[5];
    out[2] = V + (T)Da * v[3] + (T)Db * v[6];
    out[3] = E + (T)Ga * v[3] + (T)Gb * v[6];    // edge 0-1, opposite vertex 2
    out[4] = E + (T)Ga * v[1] + (T)Gb * v[4];    // edge 1-2, opposite vertex 0
    out[5] = E + (T)Ga * v[2] + (T)Gb * v[5];    // edge 2-0, opposite vertex 1
}

}  // namespace mbem
