// The FP64 pair kernels' point arithmetic compiled for the host, against long
// double: prints, per quantity, the rms error and that of a yardstick, the
// definitions evaluated in double with a square root and divisions.
#include <cmath>
#include <complex>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <random>

// the hardware's estimate: 24 bits, the rest arbitrary
static inline double host_rsq(double x) {
    double y = 1.0 / std::sqrt(x);
    uint64_t u;
    std::memcpy(&u, &y, 8);
    u ^= (u * 0x9E3779B97F4A7C15ull) >> 36;
    std::memcpy(&y, &u, 8);
    return y;
}
#define __builtin_amdgcn_rsq host_rsq
#include "../paper_2604_21181_amd/csrc/kappa64.h"
#include "../paper_2604_21181_amd/csrc/ssq_map.h"

using namespace mbem;

template <typename T>
struct Scalars {
    std::complex<T> v[5];
};
// D0, df, dg, G_eps, G_mu at R by their definitions
template <typename T>
static Scalars<T> definition(const PairConst &K, T R) {
    using C = std::complex<T>;
    const T pi4 = (T)12.566370614359172953850573533118L;
    const C k[2] = {C((T)K.ka), C((T)K.ki_re, (T)K.ki_im)};
    C phi[2], f[2], g[2];
    for (int s = 0; s < 2; ++s) {
        const C t = k[s] * R, it = C(-t.imag(), t.real());
        const T am = std::exp(-t.imag());
        const C e = C(am * std::cos(t.real()), am * std::sin(t.real()));
        phi[s] = e / (pi4 * R);
        f[s] = e * (C(3) - (T)3 * it - t * t) / (pi4 * R * R * R);
        g[s] = e * (C(1) - it) / (pi4 * R * R * R);
    }
    const C ei((T)K.eps_re, (T)K.eps_im), mi((T)K.mu_re, (T)K.mu_im);
    return {{k[0] * k[0] * phi[0] - k[1] * k[1] * phi[1], f[0] - f[1], g[0] - g[1], -R * (g[0] - ei * g[1]),
             -R * (g[0] - mi * g[1])}};
}

static void print(const char *name, double got, double yardstick, double norm) {
    std::printf("%s %.4e %.4e\n", name, std::sqrt(got / norm), std::sqrt(yardstick / norm));
}

static void scalars(double k0, double er, double ei) {
    std::complex<double> ki = k0 * std::sqrt(std::complex<double>(er, ei));
    const PairConst K = pair_const({k0, 0.0}, {ki.real(), ki.imag()}, {er, ei}, {1.0, 0.0});
    std::mt19937_64 rng(7);
    std::uniform_real_distribution<double> u(-1.0, 1.0);
    double got[5] = {}, yard[5] = {}, norm[5] = {};
    const int n = 200000;
    for (int i = 0; i < n; ++i) {
        // pairs of points of a surface: distances spread as R dR
        const double x = u(rng), y = u(rng), z = 0.1 * u(rng), d2 = x * x + y * y + z * z;
        if (K.kmax * std::sqrt(d2) < kSeriesRho) continue;
        const auto ref = definition<long double>(K, sqrtl((long double)d2));
        const auto def = definition<double>(K, std::sqrt(d2));
        const Root64 r = root64(d2);
        const KScal<double> s = scalars_closed64(K, r.r, r.inv, 1.0);
        const cx<double> v[5] = {s.D0, s.df, s.dg, s.Ge, s.Gm};
        for (int c = 0; c < 5; ++c) {
            norm[c] += (double)std::norm(ref.v[c]);
            got[c] += (double)std::norm(std::complex<long double>(v[c].re, v[c].im) - ref.v[c]);
            yard[c] += (double)std::norm(std::complex<long double>(def.v[c]) - ref.v[c]);
        }
    }
    const char *names[5] = {"D0", "df", "dg", "G_eps", "G_mu"};
    for (int c = 0; c < 5; ++c) print(names[c], got[c], yard[c], norm[c]);
}

// a P2 field of nearby nodal values (a tangent's component): the polynomial of
// p2_coef against the sum over the nodes
static void polynomial() {
    std::mt19937_64 rng(3);
    std::uniform_real_distribution<double> u(0.0, 1.0);
    double got = 0, yard = 0, norm = 0;
    const int n = 20000;
    for (int i = 0; i < n; ++i) {
        double f[6], c[6];
        const double base = 2.0 * u(rng) - 1.0;
        for (double &v : f) v = base + 0.2 * (u(rng) - 0.5);
        for (int k = 0; k < 6; ++k) c[k] = p2_coef(k, f);
        const double xi = u(rng), eta = (1.0 - xi) * u(rng);
        const double t = std::fma(c[3], xi, std::fma(c[4], eta, c[1])), s = std::fma(c[5], eta, c[2]);
        const double p = std::fma(xi, t, std::fma(eta, s, c[0]));
        auto nodes = [&](auto one) {
            using T = decltype(one);
            const T a = xi, b = eta, l = one - a - b;
            const T N[6] = {l * (2 * l - one), a * (2 * a - one), b * (2 * b - one), 4 * l * a, 4 * a * b, 4 * b * l};
            T v = 0;
            for (int k = 0; k < 6; ++k) v += N[k] * (T)f[k];
            return v;
        };
        const long double ref = nodes(1.0L);
        got += (double)((p - ref) * (p - ref));
        yard += (double)((nodes(1.0) - ref) * (nodes(1.0) - ref));
        norm += (double)(ref * ref);
    }
    print("p2", got, yard, norm);
}

int main(int argc, char **argv) {
    if (argc == 4) scalars(std::atof(argv[1]), std::atof(argv[2]), std::atof(argv[3]));
    else polynomial();
    return 0;
}
