// collide_check.cpp — host test of the collision's arithmetic
// (paper_2512_23116_amd/csrc/d3q19_mrt.hpp), run by tests/test_collide_cpu.py.
//
// accuracy  a lattice steps in FP32 (or FP64) with collide and in long double with the
//           collision written row by row from the moment matrix (App. B).  What storing
//           each population once per step in the working precision costs by itself is
//           measured too (long double collision, rounded populations).  On its way to a
//           population a value is rounded about 15 times inside the collision (pair
//           difference, momentum, s, the axis and diagonal odd parts, the sum), all of
//           the population's size, so that the error is at most sqrt(1 + 15) = 4 times
//           that of the storage.  FP32 over 4 steps (its rounded coefficients, the same
//           in every step, tell after more), FP64 over 16.
// momentum  3000 FP32 steps of a lattice with a mean flow, for several rates s_m: what
//           a step adds is rounding, without a preferred sign; 1e-9 of the momentum per
//           step (1/60 of a unit in the last place) is allowed to be one.
// rho0      lattices of any reference density and relaxation time.
#include <stdio.h>
#include <stdlib.h>

#include <cmath>
#include <initializer_list>
#include <vector>

static inline float __builtin_amdgcn_rcpf(float x) { return 1.0f / x; }
static inline float __builtin_amdgcn_sqrtf(float x) { return sqrtf(x); }
#include "d3q19_mrt.hpp"

using lbm::CollideConst;
typedef long double LD;

struct Rates {
    double e = 1.19, eps = 1.4, q = 1.2, pi = 1.4, m = 1.98;
};
static const double kTau0 = 0.51, kC = 0.13;

static CollideConst<double> constants(const Rates& r, double rho0 = 1.0, double tau0 = kTau0,
                                      double C2 = kC * kC) {
    CollideConst<double> k{};
    k.tau0 = tau0;
    k.c3 = 3.0 * C2;
    k.a_e = r.e / (38.0 * rho0);
    k.b9 = 0.5 / (tau0 * rho0);
    k.tau0_sq = tau0 * tau0;
    k.rho0 = rho0;
    lbm::fill_collide_coefficients(k, lbm::Rates{r.e, r.eps, r.q, r.pi, r.m});
    return k;
}

// eq. mrt_les_guo row by row, without a force.
static void collide_rows(LD (&g)[19], const Rates& r) {
    static LD M[19][19], norm[19];
    if (norm[0] == 0)
        for (int i = 0; i < 19; ++i) {
            const LD x = lbm::cx_of(i), y = lbm::cy_of(i), z = lbm::cz_of(i), c = x * x + y * y + z * z;
            const LD col[19] = {1, 19 * c - 30, (21 * c * c - 53 * c + 24) / 2,
                                x, (5 * c - 9) * x, y, (5 * c - 9) * y, z, (5 * c - 9) * z,
                                3 * x * x - c, (3 * c - 5) * (3 * x * x - c),
                                y * y - z * z, (3 * c - 5) * (y * y - z * z), x * y, y * z, x * z,
                                (y * y - z * z) * x, (z * z - x * x) * y, (x * x - y * y) * z};
            for (int a = 0; a < 19; ++a) {
                M[a][i] = col[a];
                norm[a] += col[a] * col[a];
            }
        }
    LD m[19], q[19] = {}, s[19];
    for (int a = 0; a < 19; ++a) {
        m[a] = 0;
        for (int i = 0; i < 19; ++i) m[a] += M[a][i] * g[i];
    }
    const LD rho = 1 + m[0], j[3] = {m[3], m[5], m[7]};
    const LD xx = j[0] * j[0] / rho, yy = j[1] * j[1] / rho, zz = j[2] * j[2] / rho;
    q[0] = m[0];
    q[1] = -11 * m[0] + 19 * (xx + yy + zz);
    q[2] = -(LD)475 / 63 * (xx + yy + zz);
    for (int a = 0; a < 3; ++a) {
        q[3 + 2 * a] = j[a];
        q[4 + 2 * a] = -(LD)2 / 3 * j[a];
    }
    q[9] = 2 * xx - yy - zz;
    q[11] = yy - zz;
    q[13] = j[0] * j[1] / rho;
    q[14] = j[1] * j[2] / rho;
    q[15] = j[0] * j[2] / rho;
    const LD n1 = m[1] - q[1], n9 = m[9] - q[9], n11 = m[11] - q[11];
    const LD s9 = 1 / (LD)kTau0;
    const LD Sxx = -(r.e * n1 + 19 * s9 * n9) / 38;
    const LD Syy = -(2 * r.e * n1 - 19 * s9 * (n9 - 3 * n11)) / 76;
    const LD Szz = -(2 * r.e * n1 - 19 * s9 * (n9 + 3 * n11)) / 76;
    LD off = 0;
    for (int a = 13; a < 16; ++a) off += (m[a] - q[a]) * (m[a] - q[a]);
    const LD S2 = 2 * (Sxx * Sxx + Syy * Syy + Szz * Szz) + 4 * (LD)2.25 * s9 * s9 * off;
    const LD nu = 1 / (kTau0 + 3 * kC * kC * sqrtl(S2));
    const LD rate[19] = {0, r.e, r.eps, 0, r.q, 0, r.q, 0, r.q, nu, r.pi, nu, r.pi, nu, nu, nu,
                         r.m, r.m, r.m};
    for (int a = 0; a < 19; ++a) s[a] = (m[a] - rate[a] * (m[a] - q[a])) / norm[a];
    for (int i = 0; i < 19; ++i) {
        g[i] = 0;
        for (int a = 0; a < 19; ++a) g[i] += M[a][i] * s[a];
    }
}

// A periodic n^3 lattice of deviations stored as R; collide is called on (R(&)[19]).
template <typename R, typename F>
static void run(std::vector<R>& f, int n, int steps, F collide) {
    const size_t N = (size_t)n * n * n;
    std::vector<R> out(19 * N);
    for (int t = 0; t < steps; ++t) {
        for (int z = 0; z < n; ++z)
            for (int y = 0; y < n; ++y)
                for (int x = 0; x < n; ++x) {
                    R g[19];
                    for (int i = 0; i < 19; ++i)
                        g[i] = f[i * N + (x - lbm::cx_of(i) + n) % n +
                                 n * ((y - lbm::cy_of(i) + n) % n + (size_t)n * ((z - lbm::cz_of(i) + n) % n))];
                    collide(g);
                    for (int i = 0; i < 19; ++i) out[i * N + x + n * (y + (size_t)n * z)] = g[i];
                }
        f.swap(out);
    }
}

// Equilibrium deviations of a mean flow U plus modes of wavenumber 1 and 2 and noise.
static std::vector<double> flow(int n, double U) {
    const size_t N = (size_t)n * n * n;
    std::vector<double> f(19 * N);
    uint64_t s = 12345;
    auto rnd = [&] { return (double)((s = s * 6364136223846793005ull + 1442695040888963407ull) >> 11) / 9007199254740992.0; };
    const double w = 2.0 * 3.14159265358979323846 / n;
    for (int z = 0; z < n; ++z)
        for (int y = 0; y < n; ++y)
            for (int x = 0; x < n; ++x) {
                const double u[3] = {U + 0.02 * sin(w * y + 1) + 0.015 * cos(2 * w * z) + 1e-3 * (2 * rnd() - 1),
                                     U + 0.02 * sin(w * z + 2) + 0.015 * cos(2 * w * x) + 1e-3 * (2 * rnd() - 1),
                                     U + 0.02 * sin(w * x + 3) + 0.015 * cos(2 * w * y) + 1e-3 * (2 * rnd() - 1)};
                const double uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
                for (int i = 0; i < 19; ++i) {
                    const double cu = lbm::cx_of(i) * u[0] + lbm::cy_of(i) * u[1] + lbm::cz_of(i) * u[2];
                    f[i * N + x + n * (y + (size_t)n * z)] =
                        (double)(float)(lbm::w_of(i) * (3 * cu + 4.5 * cu * cu - 1.5 * uu));
                }
            }
    return f;
}

// Errors of the axis, diagonal and rest populations, 2-norm against ref.
template <typename R>
static void errors(const std::vector<R>& f, const std::vector<LD>& ref, double (&e)[3]) {
    LD d[3] = {}, r[3] = {};
    const size_t N = ref.size() / 19;
    for (size_t c = 0; c < ref.size(); ++c) {
        const int i = (int)(c / N), k = i < 6 ? 0 : (i < 18 ? 1 : 2);
        d[k] += (f[c] - ref[c]) * (f[c] - ref[c]);
        r[k] += ref[c] * ref[c];
    }
    for (int k = 0; k < 3; ++k) e[k] = (double)sqrtl(d[k] / r[k]);
}

template <typename R>
static int accuracy(const Rates& r, const CollideConst<R>& k, int steps) {
    const int n = 16;
    const std::vector<double> f0 = flow(n, 0.0);
    std::vector<LD> ref(f0.begin(), f0.end());
    std::vector<R> stored(f0.begin(), f0.end()), got(f0.begin(), f0.end());
    run(ref, n, steps, [&](LD (&g)[19]) { collide_rows(g, r); });
    run(stored, n, steps, [&](R (&g)[19]) {
        LD h[19];
        for (int i = 0; i < 19; ++i) h[i] = g[i];
        collide_rows(h, r);
        for (int i = 0; i < 19; ++i) g[i] = (R)h[i];
    });
    run(got, n, steps, [&](R (&g)[19]) { lbm::collide<R>(g, R(0), R(0), R(0), k); });
    double a[3], b[3];
    errors(stored, ref, a);
    errors(got, ref, b);
    const char* name[3] = {"axis", "diagonal", "rest"};
    int bad = 0;
    for (int c = 0; c < 3; ++c) {
        printf("%s s_m %.2f, %d steps, %s: %.3g, storage alone %.3g\n", sizeof(R) == 4 ? "FP32" : "FP64",
               r.m, steps, name[c], b[c], a[c]);
        if (!(b[c] <= 4.0 * a[c])) bad = 1;
    }
    return bad;
}

static int momentum(const Rates& r) {
    const int n = 12, steps = 3000;
    const std::vector<double> f0 = flow(n, 0.03);
    std::vector<float> f(f0.begin(), f0.end());
    const CollideConst<float> k = lbm::round_constants(constants(r));
    run(f, n, steps, [&](float (&g)[19]) { lbm::collide<float>(g, 0.f, 0.f, 0.f, k); });
    const size_t N = (size_t)n * n * n;
    int bad = 0;
    for (int a = 0; a < 3; ++a) {
        double before = 0, after = 0;
        for (size_t c = 0; c < 19 * N; ++c) {
            const int i = (int)(c / N), v = a == 0 ? lbm::cx_of(i) : (a == 1 ? lbm::cy_of(i) : lbm::cz_of(i));
            before += v * f0[c];
            after += v * (double)f[c];
        }
        const double drift = after / before - 1.0;
        printf("s_m %.2f: momentum %d drifts by %.2e in %d steps\n", r.m, a, drift, steps);
        if (!(fabs(drift) <= 1e-9 * steps)) bad = 1;
    }
    return bad;
}

// The collision of rho0 2^n and populations times 2^n is 2^n times that of rho0; the
// factors of two round nowhere, those of the rescaled strain norm apart (three roundings
// of tau_e - tau0 more, which is a tenth of tau_e at most here).
template <typename R>
static int scaled(const Rates& r, std::initializer_list<int> powers,
                  CollideConst<R> (*constants_of)(const CollideConst<double>&)) {
    const int n = 8;
    const double unit = sizeof(R) == 4 ? 6e-8 : 1.2e-16;
    const std::vector<double> f0 = flow(n, 0.01);
    int bad = 0;
    for (int p : powers) {
        double worst = 0, most = 0;
        const CollideConst<R> k0 = constants_of(constants(r, 1.0, kTau0, 4.0));
        const CollideConst<R> k1 = constants_of(constants(r, ldexp(1.0, p), kTau0, 4.0));
        std::vector<R> a(f0.begin(), f0.end()), b(a);
        for (R& v : b) v = (R)ldexp((double)v, p);
        run(a, n, 4, [&](R (&g)[19]) { lbm::collide<R>(g, R(0), R(0), R(0), k0); });
        run(b, n, 4, [&](R (&g)[19]) { lbm::collide<R>(g, R(0), R(0), R(0), k1); });
        for (size_t c = 0; c < a.size(); ++c) {
            worst = fmax(worst, fabs(ldexp((double)b[c], -p) - a[c]));
            most = fmax(most, fabs((double)a[c]));
        }
        printf("rho0 = 2^%d: %.2e of the populations off those of rho0 = 1\n", p, worst / most);
        if (!(worst <= 4 * 3 * unit * most)) bad = 1;
    }
    // a tau0 whose square leaves the type: the shear rows keep all but 1/tau0 of themselves
    for (double tau0 : {1e22, 1e37, sizeof(R) == 4 ? 3e38 : 1e300}) {
        const CollideConst<R> k = constants_of(constants(r, 1.0, tau0, 4.0));
        std::vector<R> a(f0.begin(), f0.end()), b(f0.size(), R(0));
        run(a, n, 2, [&](R (&g)[19]) { lbm::collide<R>(g, R(0), R(0), R(0), k); });
        run(b, n, 2, [&](R (&g)[19]) { lbm::collide<R>(g, R(0), R(0), R(0), k); });   // at rest
        for (R v : a)
            if (!std::isfinite(v)) bad = 1;
        for (R v : b)
            if (v != 0) bad = 1;
        if (bad) printf("tau0 = %g\n", tau0);
    }
    return bad;
}
static CollideConst<double> unrounded(const CollideConst<double>& k) { return k; }

int main(int argc, char** argv) {
    if (argc != 3) return 2;
    Rates r;
    r.m = atof(argv[2]);
    const CollideConst<double> k = constants(r);
    switch (argv[1][0]) {
        case 's': return accuracy<float>(r, lbm::round_constants(k), 4);
        case 'd': return accuracy<double>(r, k, 16);
        case 'm': return momentum(r);
        case 'r':
            return scaled<float>(r, {-90, -70, -45, -20, 20, 40, 70, 100}, lbm::round_constants) |
                   scaled<double>(r, {-700, -400, 400, 700}, unrounded);
    }
    return 2;
}
