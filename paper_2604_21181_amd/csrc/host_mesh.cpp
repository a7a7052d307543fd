// Host preprocessing of a P2 surface mesh: topology validation, the double
// Morton permutation of Sec. 5, renumbering, node incidence, singular
// element-pair lists (Sec. 4.2) and the sparsity pattern of the mass matrix.
#include <algorithm>
#include <cmath>
#include <map>
#include <numeric>
#include <unordered_map>

#include "mbem_internal.h"

namespace mbem {

namespace {

// Spread the low 21 bits of v so that bit b lands on bit 3b.
inline uint64_t spread_bits3(uint64_t v) {
    v &= 0x1fffffULL;
    v = (v | (v << 32)) & 0x1f00000000ffffULL;
    v = (v | (v << 16)) & 0x1f0000ff0000ffULL;
    v = (v | (v << 8)) & 0x100f00f00f00f00fULL;
    v = (v | (v << 4)) & 0x10c30c30c30c30c3ULL;
    v = (v | (v << 2)) & 0x1249249249249249ULL;
    return v;
}

inline uint64_t quantise(double x, double lo, double ext) {
    double q = std::floor((x - lo) / ext * 2097152.0);  // 2^21 cells per side
    if (q < 0.0) q = 0.0;
    if (q > 2097151.0) q = 2097151.0;
    return (uint64_t)q;
}

inline uint64_t zorder(const double p[3], const double lo[3], double ext) {
    return spread_bits3(quantise(p[0], lo[0], ext)) |
           (spread_bits3(quantise(p[1], lo[1], ext)) << 1) |
           (spread_bits3(quantise(p[2], lo[2], ext)) << 2);
}

std::vector<int64_t> stable_order(const std::vector<uint64_t> &key) {
    std::vector<int64_t> ord(key.size());
    std::iota(ord.begin(), ord.end(), 0);
    std::stable_sort(ord.begin(), ord.end(),
                     [&](int64_t a, int64_t b) { return key[a] < key[b]; });
    return ord;
}

}  // namespace

int morton_order_host(const double *xyz, int64_t nn, const int64_t *tri6,
                      int64_t nt, std::vector<int64_t> &node_order,
                      std::vector<int64_t> &tri_order, std::vector<uint64_t> *node_keys) {
    for (int64_t i = 0; i < 3 * nn; ++i)
        if (!std::isfinite(xyz[i])) {
            set_error("node coordinate " + std::to_string(i) + " is not finite");
            return MBEM_EINVAL;
        }
    double lo[3], hi[3];
    for (int d = 0; d < 3; ++d) lo[d] = hi[d] = xyz[d];
    for (int64_t v = 0; v < nn; ++v)
        for (int d = 0; d < 3; ++d) {
            lo[d] = std::min(lo[d], xyz[3 * v + d]);
            hi[d] = std::max(hi[d], xyz[3 * v + d]);
        }
    double ext = std::max(hi[0] - lo[0], std::max(hi[1] - lo[1], hi[2] - lo[2]));
    if (!(ext > 0.0)) {
        set_error("degenerate mesh bounding box");
        return MBEM_EMESH;
    }
    std::vector<uint64_t> key(nn);
    for (int64_t v = 0; v < nn; ++v) key[v] = zorder(xyz + 3 * v, lo, ext);
    node_order = stable_order(key);
    if (node_keys) {
        node_keys->resize(nn);
        for (int64_t k = 0; k < nn; ++k) (*node_keys)[k] = key[node_order[k]];
    }
    key.assign(nt, 0);
    for (int64_t t = 0; t < nt; ++t) {
        double c[3];
        for (int d = 0; d < 3; ++d) {
            double s = xyz[3 * tri6[6 * t] + d] + xyz[3 * tri6[6 * t + 1] + d];
            s = s + xyz[3 * tri6[6 * t + 2] + d];
            c[d] = s / 3.0;
        }
        key[t] = zorder(c, lo, ext);
    }
    tri_order = stable_order(key);
    return MBEM_OK;
}

// Legendre roots and weights on [-1, 1] by Newton iteration.
void gauss_legendre(int n, double *x, double *w) {
    const double pi = 3.14159265358979323846;
    for (int i = 0; i < n; ++i) {
        double z = std::cos(pi * (i + 0.75) / (n + 0.5));
        double pn = 0, dpn = 1;
        for (int it = 0; it < 200; ++it) {
            double pm = 1.0, pc = z;             // P_0, P_1
            for (int k = 2; k <= n; ++k) {
                double pk = ((2 * k - 1) * z * pc - (k - 1) * pm) / k;
                pm = pc;
                pc = pk;
            }
            pn = (n == 1) ? z : pc;
            double pprev = (n == 1) ? 1.0 : pm;
            dpn = n * (pprev - z * pn) / (1.0 - z * z);
            double dz = pn / dpn;
            z -= dz;
            if (std::fabs(dz) < 1e-16) break;
        }
        {
            double pm = 1.0, pc = z;
            for (int k = 2; k <= n; ++k) {
                double pk = ((2 * k - 1) * z * pc - (k - 1) * pm) / k;
                pm = pc;
                pc = pk;
            }
            pn = (n == 1) ? z : pc;
            double pprev = (n == 1) ? 1.0 : pm;
            dpn = n * (pprev - z * pn) / (1.0 - z * z);
        }
        x[i] = z;
        w[i] = 2.0 / ((1.0 - z * z) * dpn * dpn);
    }
}

int build_mesh_host(const double *xyz_in, int64_t nn, const int64_t *tri_in,
                    int64_t nt, mbem_mesh *m) {
    if (nn < 4 || nt < 4 || nn > (1LL << 29) || nt > (1LL << 28)) {
        set_error("mesh sizes out of range");
        return MBEM_EINVAL;
    }
    // ---- index checks and vertex / mid-edge roles
    std::vector<int8_t> role(nn, 0);  // 1 vertex, 2 mid-edge
    for (int64_t t = 0; t < nt; ++t)
        for (int k = 0; k < 6; ++k) {
            int64_t v = tri_in[6 * t + k];
            if (v < 0 || v >= nn) {
                set_error("triangle node index out of range");
                return MBEM_EINVAL;
            }
            int8_t r = k < 3 ? 1 : 2;
            if (role[v] && role[v] != r) {
                set_error("node used both as a vertex and as a mid-edge node");
                return MBEM_EMESH;
            }
            role[v] = r;
            for (int l = 0; l < k; ++l)
                if (tri_in[6 * t + l] == v) {
                    set_error("repeated node inside a triangle");
                    return MBEM_EMESH;
                }
        }
    for (int64_t v = 0; v < nn; ++v)
        if (!role[v]) {
            set_error("node not referenced by any triangle");
            return MBEM_EMESH;
        }
    // ---- every edge in exactly two triangles, opposite directions, one mid
    struct EdgeUse { int64_t t; int a; bool fwd; int64_t mid; };
    std::unordered_map<uint64_t, std::vector<EdgeUse>> edges;
    edges.reserve(3 * nt);
    for (int64_t t = 0; t < nt; ++t)
        for (int a = 0; a < 3; ++a) {
            int64_t u = tri_in[6 * t + a], v = tri_in[6 * t + (a + 1) % 3];
            uint64_t key = (uint64_t)std::min(u, v) << 32 | (uint64_t)std::max(u, v);
            edges[key].push_back({t, a, u < v, tri_in[6 * t + 3 + a]});
        }
    for (auto &kv : edges) {
        const auto &u = kv.second;
        if (u.size() != 2 || u[0].fwd == u[1].fwd || u[0].mid != u[1].mid) {
            set_error("mesh is not a closed, consistently oriented P2 surface");
            return MBEM_EMESH;
        }
    }
    // ---- Morton permutation and renumbering
    std::vector<int64_t> no, to;
    MBEM_TRY(morton_order_host(xyz_in, nn, tri_in, nt, no, to, &m->node_key));
    std::vector<int64_t> rank(nn);
    for (int64_t k = 0; k < nn; ++k) rank[no[k]] = k;
    m->nn = nn;
    m->nt = nt;
    m->node_order = no;
    m->tri_order = to;
    m->xyz.resize(3 * nn);
    m->amax = 0.0;
    for (int64_t k = 0; k < nn; ++k) {
        double r2 = 0;
        for (int d = 0; d < 3; ++d) {
            m->xyz[3 * k + d] = xyz_in[3 * no[k] + d];
            r2 += m->xyz[3 * k + d] * m->xyz[3 * k + d];
        }
        m->amax = std::max(m->amax, std::sqrt(r2));
    }
    m->tri.resize(6 * nt);
    for (int64_t t = 0; t < nt; ++t)
        for (int k = 0; k < 6; ++k)
            m->tri[6 * t + k] = (int32_t)rank[tri_in[6 * to[t] + k]];
    return MBEM_OK;
}

}  // namespace mbem

// ------------------------------------------------------------------------
// incidence, singular pairs and mass pattern on the renumbered mesh
// ------------------------------------------------------------------------
namespace mbem {

// perm code: three 2-bit local vertex indices (re-indexed order)
static inline int32_t pack_perm(int a, int b, int c) { return a | (b << 2) | (c << 4); }

// Test batches per band of the FP64 regular-pair fill.  The two band buffers
// together stay below kPairScratch where a band has more than one batch, so
// that they are written and read back while in the 256 MB last-level cache.  A
// band is at least one batch, whose two buffers grow with the mesh: 224 MB at
// 9 400 triangles, 290 MB at 12 300, written through to memory from there on
// (9 408 triangles, fill 238 ms where the colour classes took 628).  Of the bands
// that fit, the largest is cut towards whole rounds of 768 workgroups (three
// per compute unit; node-attached tangents run two), rounded down to whole
// batches: 1.95 rounds at 320 triangles, 1.7 at 1280, 1.6 at 3072, what one batch
// has from 5120 on.
constexpr int64_t kPairScratch = (int64_t)224 << 20, kPairRound = 768;

static int64_t pair_band(int64_t nbatch, int64_t nslots) {
    const int64_t per = 6 * 2 * 16 * nslots * nslots / nbatch;      // bytes per test batch, on average
    if (nbatch * per <= kPairScratch / 2) return nbatch;            // a single band
    int64_t band = std::max<int64_t>(1, kPairScratch / 2 / per);
    const int64_t rounds = band * nbatch / kPairRound;
    if (rounds > 0) band = std::max<int64_t>(1, rounds * kPairRound / nbatch);
    return band;
}

int build_tables(const mbem_mesh *m, MeshTables &T) {
    const int64_t nn = m->nn, nt = m->nt;
    const int32_t *tri = m->tri.data();
    // node incidence
    T.inc_ptr.assign(nn + 1, 0);
    for (int64_t t = 0; t < nt; ++t)
        for (int k = 0; k < 6; ++k) T.inc_ptr[tri[6 * t + k] + 1]++;
    for (int64_t v = 0; v < nn; ++v) T.inc_ptr[v + 1] += T.inc_ptr[v];
    T.inc.assign(T.inc_ptr[nn], 0);
    {
        std::vector<int32_t> fill(T.inc_ptr.begin(), T.inc_ptr.end() - 1);
        for (int64_t t = 0; t < nt; ++t)
            for (int k = 0; k < 6; ++k) T.inc[fill[tri[6 * t + k]]++] = (int32_t)(t * 8 + k);
    }
    // singular pairs: for every test triangle e, all triangles f sharing at
    // least one vertex node, with both re-indexed so that the shared
    // vertices come first, ordered along e's counter-clockwise edge.
    std::vector<int32_t> cand;
    for (int64_t e = 0; e < nt; ++e) {
        cand.clear();
        for (int a = 0; a < 3; ++a) {
            int32_t v = tri[6 * e + a];
            for (int32_t s = T.inc_ptr[v]; s < T.inc_ptr[v + 1]; ++s)
                if ((T.inc[s] & 7) < 3) cand.push_back(T.inc[s] >> 3);
        }
        std::sort(cand.begin(), cand.end());
        cand.erase(std::unique(cand.begin(), cand.end()), cand.end());
        for (int32_t f : cand) {
            int pos_e[3], pos_f[3], ns = 0;
            for (int a = 0; a < 3; ++a)
                for (int b = 0; b < 3; ++b)
                    if (tri[6 * e + a] == tri[6 * f + b]) { pos_e[ns] = a; pos_f[ns] = b; ++ns; }
            int32_t pe, pf;
            if (ns == 3) {
                pe = pf = pack_perm(0, 1, 2);
            } else if (ns == 2) {
                // A -> B must be an edge of e in e's own orientation
                int i0 = 0, i1 = 1;
                if ((pos_e[0] + 1) % 3 != pos_e[1]) { i0 = 1; i1 = 0; }
                int ea = pos_e[i0], eb = pos_e[i1], fa = pos_f[i0], fb = pos_f[i1];
                pe = pack_perm(ea, eb, 3 - ea - eb);
                pf = pack_perm(fa, fb, 3 - fa - fb);
            } else {
                pe = pack_perm(pos_e[0], (pos_e[0] + 1) % 3, (pos_e[0] + 2) % 3);
                pf = pack_perm(pos_f[0], (pos_f[0] + 1) % 3, (pos_f[0] + 2) % 3);
            }
            T.spairs.push_back((int32_t)e);
            T.spairs.push_back(f);
            T.spairs.push_back(ns);
            T.spairs.push_back(pe | (pf << 6));
            T.n_single[ns]++;
        }
    }
    // mass pattern: nodes sharing a triangle
    T.m_ptr.assign(nn + 1, 0);
    T.m_col.clear();
    {
        std::vector<int32_t> seen(nn, -1);
        for (int64_t v = 0; v < nn; ++v) {
            const size_t at = T.m_col.size();
            for (int32_t s = T.inc_ptr[v]; s < T.inc_ptr[v + 1]; ++s)
                for (int l = 0; l < 6; ++l) {
                    const int32_t u = tri[6 * (int64_t)(T.inc[s] >> 3) + l];
                    if (seen[u] == v) continue;
                    seen[u] = (int32_t)v;
                    T.m_col.push_back(u);
                }
            std::sort(T.m_col.begin() + at, T.m_col.end());
            T.m_ptr[v + 1] = (int32_t)T.m_col.size();
        }
    }
    T.m_slot.resize(36 * nt);
    for (int64_t t = 0; t < nt; ++t)
        for (int k = 0; k < 6; ++k)
            for (int l = 0; l < 6; ++l) {
                int32_t i = tri[6 * t + k], j = tri[6 * t + l];
                auto b = T.m_col.begin() + T.m_ptr[i], en = T.m_col.begin() + T.m_ptr[i + 1];
                T.m_slot[36 * t + 6 * k + l] = (int32_t)(std::lower_bound(b, en, j) - T.m_col.begin());
            }
    // trial chunks: kChunk Morton-consecutive triangles, their distinct
    // nodes ("slots", ascending) and, per slot, the (triangle, local node)
    // pairs that touch it
    const int64_t nch = (nt + kChunk - 1) / kChunk;
    T.chunks.assign(nch * kChunkRec, 0);
    std::vector<std::pair<int32_t, int32_t>> uses;   // (node, local triangle * 8 + loc)
    for (int64_t k = 0; k < nch; ++k) {
        int32_t *rec = T.chunks.data() + k * kChunkRec;
        uses.clear();
        for (int fs = 0; fs < kChunk; ++fs) {
            const int64_t f = k * kChunk + fs;
            if (f >= nt) break;
            for (int l = 0; l < 6; ++l) uses.push_back({tri[6 * f + l], fs * 8 + l});
        }
        std::sort(uses.begin(), uses.end());
        int ns = 0, ni = 0;
        for (size_t u = 0; u < uses.size(); ++u) {
            if (u == 0 || uses[u].first != uses[u - 1].first) {
                rec[1 + ns] = uses[u].first;
                rec[25 + ns] = ni;
                ++ns;
            }
            rec[50 + ni] = uses[u].second;
            ++ni;
        }
        rec[0] = ns;
        rec[25 + ns] = ni;
    }
    // column ranges: L.rng consecutive nodes; the triangles touching a
    // range (ascending) in batches of L.nb, and per batch the incidences of
    // the range's nodes grouped by node
    {
        constexpr RngLayout L = kRng;
        std::vector<int32_t> &off = T.rng_off, &recs = T.rng_rec;
        const int64_t nrng = (nn + L.rng - 1) / L.rng;
        off.assign(nrng + 1, 0);
        recs.clear();
        std::vector<int32_t> rtris;
        for (int64_t r = 0; r < nrng; ++r) {
            const int64_t j0 = r * L.rng, j1 = std::min<int64_t>(nn, j0 + L.rng);
            rtris.clear();
            for (int64_t j = j0; j < j1; ++j)
                for (int32_t q = T.inc_ptr[j]; q < T.inc_ptr[j + 1]; ++q) rtris.push_back(T.inc[q] >> 3);
            std::sort(rtris.begin(), rtris.end());
            rtris.erase(std::unique(rtris.begin(), rtris.end()), rtris.end());
            for (size_t b0 = 0; b0 < rtris.size(); b0 += L.nb) {
                const size_t base = recs.size();
                recs.resize(base + L.rec(), 0);
                int32_t *rec = recs.data() + base;
                const int nb = (int)std::min<size_t>(L.nb, rtris.size() - b0);
                uses.clear();            // (range-local node, fb*8 + loc)
                rec[0] = nb;
                for (int fb = 0; fb < nb; ++fb) {
                    const int32_t f = rtris[b0 + fb];
                    rec[1 + fb] = f;
                    for (int l = 0; l < 6; ++l) {
                        const int32_t v = tri[6 * (int64_t)f + l];
                        if (v >= j0 && v < j1) uses.push_back({(int32_t)(v - j0), fb * 8 + l});
                    }
                }
                std::sort(uses.begin(), uses.end());
                size_t u = 0;
                for (int jl = 0; jl <= L.rng; ++jl) {
                    while (u < uses.size() && uses[u].first < jl) ++u;
                    rec[L.off() + jl] = (int32_t)u;
                }
                for (size_t k = 0; k < uses.size(); ++k) rec[L.inc() + k] = uses[k].second;
            }
            off[r + 1] = (int32_t)(recs.size() / L.rec());
        }
    }
    // Trial batches of the FP64 regular-pair fill: grown from the first free
    // triangle (Morton order) by the free neighbour that shares the most
    // nodes with the batch, and among those the one with the fewest free
    // neighbours of its own, so that few triangles are left alone; without a
    // neighbour that fits, the next free triangle that fits.  About 18 nodes
    // per 5 triangles (20.4 for runs of the Morton order).
    {
        std::vector<char> used(nt, 0);
        // per row of the scratch, in order: its node and its place in the records
        std::vector<int32_t> row_node, row_place;
        row_node.reserve(4 * nt);
        row_place.reserve(4 * nt);
        T.pair_rec.reserve((nt / 4 + 1) * kPairRec);
        int32_t nodes = 0;
        // edge neighbours, and the batch that last held a node / listed a triangle
        std::vector<int32_t> nbr(3 * nt), in_batch(nn, -1), listed(nt, -1);
        for (int64_t t = 0; t < nt; ++t)
            for (int k = 0; k < 3; ++k) {
                const int32_t mid = tri[6 * t + 3 + k];
                nbr[3 * t + k] = (int32_t)t;
                for (int32_t q = T.inc_ptr[mid]; q < T.inc_ptr[mid + 1]; ++q)
                    if ((T.inc[q] >> 3) != t) nbr[3 * t + k] = T.inc[q] >> 3;
            }
        std::vector<int32_t> bt, bn, cand;     // the batch's triangles and nodes, triangles around them
        std::vector<std::pair<int, int32_t>> order;
        int32_t id = 0;
        auto shared = [&](int32_t f) {
            int n = 0;
            for (int k = 0; k < 6; ++k) n += in_batch[tri[6 * (int64_t)f + k]] == id;
            return n;
        };
        auto fits = [&](int n) { return (int)bn.size() + 6 - n <= kPairNS; };
        auto add = [&](int32_t f) {
            used[f] = 1;
            bt.push_back(f);
            for (int k = 0; k < 6; ++k) {
                const int32_t v = tri[6 * (int64_t)f + k];
                if (in_batch[v] == id) continue;
                in_batch[v] = id;
                bn.push_back(v);
                for (int32_t s = T.inc_ptr[v]; s < T.inc_ptr[v + 1]; ++s) {
                    const int32_t c = T.inc[s] >> 3;
                    if (used[c] || listed[c] == id) continue;
                    listed[c] = id;
                    cand.push_back(c);
                }
            }
        };
        for (int64_t first = 0;; ++id) {
            while (first < nt && used[first]) ++first;
            if (first == nt) break;
            bt.clear();
            bn.clear();
            cand.clear();
            add((int32_t)first);
            while ((int)bt.size() < kPairNB) {
                int32_t best = -1;
                int best_score = -1;
                for (int32_t f : cand) {
                    if (used[f]) continue;
                    const int n = shared(f);
                    if (!fits(n)) continue;
                    const int score = 4 * n + used[nbr[3 * f]] + used[nbr[3 * f + 1]] + used[nbr[3 * f + 2]];
                    if (score > best_score || (score == best_score && f < best)) { best_score = score; best = f; }
                }
                if (best < 0)
                    for (int64_t f = first + 1; f < std::min(nt, first + 64) && best < 0; ++f)
                        if (!used[f] && fits(shared((int32_t)f))) best = (int32_t)f;
                if (best < 0) break;
                add(best);
            }
            std::sort(bt.begin(), bt.end());
            // nodes by falling number of incidences in the batch
            order.clear();
            for (int32_t v : bn) {
                int n = 0;
                for (int32_t f : bt)
                    for (int l = 0; l < 6; ++l) n += tri[6 * (int64_t)f + l] == v;
                order.push_back({-n, v});
            }
            std::sort(order.begin(), order.end());
            for (size_t q = 0; q < bn.size(); ++q) bn[q] = order[q].second;
            const size_t base = T.pair_rec.size();
            T.pair_rec.resize(base + kPairRec, 0);
            int32_t *rec = T.pair_rec.data() + base;
            rec[0] = (int32_t)bt.size();
            rec[1] = (int32_t)bn.size();
            rec[2] = nodes;
            T.pair_row0.push_back(nodes);
            for (size_t k = 0; k < bt.size(); ++k) rec[kPairTri + k] = bt[k];
            int ni = 0;
            for (size_t q = 0; q < bn.size(); ++q) {
                rec[kPairOff + q] = ni;
                bool seen = false;
                for (size_t k = 0; k < bt.size(); ++k)
                    for (int l = 0; l < 6; ++l)
                        if (tri[6 * (int64_t)bt[k] + l] == bn[q]) {
                            rec[kPairInc + ni++] = (int32_t)(8 * k + l);
                            rec[kPairLoc + 6 * k + l] = (int32_t)q + (seen ? 0 : 256);
                            seen = true;
                        }
                row_node.push_back(bn[q]);
                row_place.push_back((int32_t)(base + kPairPos + q));
            }
            rec[kPairOff + bn.size()] = ni;
            nodes += (int32_t)bn.size();
        }
        T.pair_sptr.assign(nn + 1, 0);
        for (int32_t v : row_node) ++T.pair_sptr[v + 1];
        for (int64_t v = 0; v < nn; ++v) T.pair_sptr[v + 1] += T.pair_sptr[v];
        T.pair_srow.resize(nodes);
        std::vector<int32_t> next(T.pair_sptr.begin(), T.pair_sptr.end() - 1);
        for (int32_t row = 0; row < nodes; ++row) {
            const int32_t slot = next[row_node[row]]++;
            T.pair_rec[row_place[row]] = slot;
            T.pair_srow[slot] = row;
        }
        T.pair_cb.assign(1, 0);
        for (int64_t v = 0; v < nn; ++v)
            if (v > T.pair_cb.back() && T.pair_sptr[v + 1] - T.pair_sptr[T.pair_cb.back()] > kPairCols)
                T.pair_cb.push_back((int32_t)v);
        T.pair_cb.push_back((int32_t)nn);
        const int64_t nbatch = (int64_t)T.pair_row0.size();
        T.pair_row0.push_back(nodes);
        T.pair_band = pair_band(nbatch, nodes);
        const int64_t nbands = (nbatch + T.pair_band - 1) / T.pair_band;
        std::vector<int32_t> band_end;       // first node row after each band
        for (int64_t b = 0; b < nbands; ++b) band_end.push_back(T.pair_row0[std::min(nbatch, (b + 1) * T.pair_band)]);
        std::vector<std::vector<int32_t>> tasks(nbands);
        for (int64_t v = 0; v < nn; ++v) {
            const int32_t s1 = T.pair_sptr[v + 1];
            for (int32_t s = T.pair_sptr[v]; s < s1;) {
                const int64_t b = std::upper_bound(band_end.begin(), band_end.end(), T.pair_srow[s]) - band_end.begin();
                int32_t q = s;
                while (q < s1 && T.pair_srow[q] < band_end[b]) ++q;
                for (int32_t x : {(int32_t)v, s, q, (int32_t)(s == T.pair_sptr[v])}) tasks[b].push_back(x);
                s = q;
            }
        }
        T.pair_rows_off.assign(1, 0);
        for (auto &t : tasks) {
            T.pair_rows.insert(T.pair_rows.end(), t.begin(), t.end());
            T.pair_rows_off.push_back((int64_t)T.pair_rows.size() / 4);
        }
    }
    // Colour classes (greedy in Morton order, then balanced) so that the
    // regular-pair fill can add to Z with plain read-modify-write: inside one
    // launch no two test triangles share a node (disjoint rows) and no two
    // trial chunks share a node (disjoint columns).  Balancing moves items from classes above the mean
    // size to smaller classes they do not conflict with, so that every
    // launch has about the same number of workgroups.
    auto colour = [&](int64_t nitems, auto nodes_of, std::vector<int32_t> &list,
                      std::vector<int32_t> &off) {
        std::vector<std::vector<int32_t>> users(nn);
        std::vector<int32_t> item_nodes, first(1, 0);    // an item's nodes: [first[it], first[it + 1])
        item_nodes.reserve(6 * nt);
        std::vector<int32_t> col(nitems, -1);
        std::vector<int64_t> used(1, -1);    // colour -> the last item (or pass and item) that met it
        int ncol = 0;
        for (int64_t it = 0; it < nitems; ++it) {
            nodes_of(it, item_nodes);
            first.push_back((int32_t)item_nodes.size());
            for (int32_t k = first[it]; k < first[it + 1]; ++k)
                for (int32_t o : users[item_nodes[k]]) used[col[o]] = it;
            int c = 0;
            while (c < ncol && used[c] == it) ++c;
            if (c == ncol) used.push_back(-1);
            col[it] = c;
            ncol = std::max(ncol, c + 1);
            for (int32_t k = first[it]; k < first[it + 1]; ++k) users[item_nodes[k]].push_back((int32_t)it);
        }
        std::vector<int64_t> size(ncol, 0);
        for (int64_t it = 0; it < nitems; ++it) size[col[it]]++;
        const int64_t target = (nitems + ncol - 1) / ncol;
        for (int round = 0; round < 8; ++round) {
            int64_t moved = 0;
            for (int64_t it = 0; it < nitems; ++it) {
                const int c = col[it];
                if (size[c] <= target) continue;
                const int64_t mark = (round + 1) * nitems + it;
                for (int32_t k = first[it]; k < first[it + 1]; ++k)
                    for (int32_t o : users[item_nodes[k]])
                        if (o != it) used[col[o]] = mark;
                int best = -1;
                for (int d = 0; d < ncol; ++d)
                    if (used[d] != mark && size[d] < target && (best < 0 || size[d] < size[best])) best = d;
                if (best >= 0) { col[it] = best; --size[c]; ++size[best]; ++moved; }
            }
            if (!moved) break;
        }
        off.assign(ncol + 1, 0);
        for (int64_t it = 0; it < nitems; ++it) off[col[it] + 1]++;
        for (int c = 0; c < ncol; ++c) off[c + 1] += off[c];
        list.assign(nitems, 0);
        std::vector<int32_t> fill(off.begin(), off.end() - 1);
        for (int64_t it = 0; it < nitems; ++it) list[fill[col[it]]++] = (int32_t)it;
    };
    colour(nt, [&](int64_t e, std::vector<int32_t> &out) {
        for (int k = 0; k < 6; ++k) out.push_back(tri[6 * e + k]);
    }, T.tcol_list, T.tcol_off);
    {
        // the triangles of a node have distinct test colours: the lowest one
        // writes the node's rows first
        std::vector<int32_t> tcolour(nt), low(nn, INT32_MAX);
        for (size_t c = 0; c + 1 < T.tcol_off.size(); ++c)
            for (int32_t q = T.tcol_off[c]; q < T.tcol_off[c + 1]; ++q) tcolour[T.tcol_list[q]] = (int32_t)c;
        for (int64_t e = 0; e < nt; ++e)
            for (int k = 0; k < 6; ++k) low[tri[6 * e + k]] = std::min(low[tri[6 * e + k]], tcolour[e]);
        T.row_first.assign(nt, 0);
        for (int64_t e = 0; e < nt; ++e)
            for (int k = 0; k < 6; ++k)
                if (tcolour[e] == low[tri[6 * e + k]]) T.row_first[e] |= 1 << k;
    }
    colour(nch, [&](int64_t k, std::vector<int32_t> &out) {
        const int32_t *rec = T.chunks.data() + k * kChunkRec;
        for (int s2 = 0; s2 < rec[0]; ++s2) out.push_back(rec[1 + s2]);
    }, T.ccol_list, T.ccol_off);
    {
        // likewise the chunks of a node: the lowest chunk colour writes the
        // node's columns first
        std::vector<int32_t> ccolour(nch), low(nn, INT32_MAX);
        for (size_t c = 0; c + 1 < T.ccol_off.size(); ++c)
            for (int32_t q = T.ccol_off[c]; q < T.ccol_off[c + 1]; ++q) ccolour[T.ccol_list[q]] = (int32_t)c;
        for (int64_t k = 0; k < nch; ++k) {
            const int32_t *rec = T.chunks.data() + k * kChunkRec;
            for (int s2 = 0; s2 < rec[0]; ++s2) low[rec[1 + s2]] = std::min(low[rec[1 + s2]], ccolour[k]);
        }
        T.col_first.assign(nch, 0);
        for (int64_t k = 0; k < nch; ++k) {
            const int32_t *rec = T.chunks.data() + k * kChunkRec;
            for (int s2 = 0; s2 < rec[0]; ++s2)
                if (ccolour[k] == low[rec[1 + s2]]) T.col_first[k] |= 1 << s2;
        }
    }
    return MBEM_OK;
}

}  // namespace mbem
