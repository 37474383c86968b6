// d3q19_mrt.hpp — per-cell D3Q19 MRT-Smagorinsky-Guo collision for gfx950.
//
// One thread owns one cell.  Populations are deviations g = f - w rho0, whose
// moments are M f - rho0 (1, -11, 3, 0, ..., 0) (App. B eq. moment-matrix); the
// equilibrium moments of eq. meq_fm are printed in exactly that deviation form
// (row 0 is delta rho).  Two functions:
//   cell_macro  density, velocity and tau_e of a cell (diagnostics);
//   collide     the whole collision of the step kernels, in place.
// Both split every opposite pair (2k, 2k+1) into its sum p_k, which alone
// enters the even-parity rows (0, 1, 2, 9..15), and its difference d_k, which
// alone enters the odd-parity rows (3..8, 16..18).
#pragma once

#include <float.h>
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <stdlib.h>

namespace lbm {

// Velocity set of App. B Fig. d3q19_table (0-based, rest = 18).
__host__ __device__ constexpr int cx_of(int i) {
    constexpr int v[19] = {1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 0};
    return v[i];
}
__host__ __device__ constexpr int cy_of(int i) {
    constexpr int v[19] = {0, 0, 1, -1, 0, 0, 1, -1, -1, 1, 1, -1, 1, -1, 0, 0, 0, 0, 0};
    return v[i];
}
__host__ __device__ constexpr int cz_of(int i) {
    constexpr int v[19] = {0, 0, 0, 0, 1, -1, 0, 0, 0, 0, 1, -1, -1, 1, 1, -1, -1, 1, 0};
    return v[i];
}
__host__ __device__ constexpr int opp_of(int i) { return i == 18 ? 18 : (i ^ 1); }
__host__ __device__ constexpr double w_of(int i) {
    return i < 6 ? 1.0 / 18.0 : (i < 18 ? 1.0 / 36.0 : 1.0 / 3.0);
}

// Reciprocal and square root: hardware v_rcp_f32 / v_sqrt_f32 (1 ulp) in FP32,
// IEEE operations in FP64.
__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double fast_rcp(double x) { return 1.0 / x; }
__device__ __forceinline__ float fast_sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
__device__ __forceinline__ double fast_sqrt(double x) { return sqrt(x); }

// Bits of CollideConst::closure, 0 for the usual lattice.
constexpr int32_t kSelfConsistent = 1;   // s_9 = 1/tau_e in eq. yu_strain, closed form
constexpr int32_t kRescaled = 2;         // collide divides the moments of the strain norm by
constexpr int32_t kScaleShift = 8;       // 2^(closure >> kScaleShift)

// Constants of one lattice's collision, in the arithmetic type R.  Those that collide
// reads come first, 92 bytes in FP32 (see LatticeArgs); cell_macro and the derivation
// read the rest.
template <typename R>
struct CollideConst {
    R tau0;      // bare relaxation time
    R rho0;
    R tau0_sq;   // tau0^2
    int32_t closure;           // kSelfConsistent, kRescaled and its exponent
    // coefficients of collide, formed in FP64 by fill_collide_coefficients
    R ea_sa, ea_sd, ea_r, ea_u2, ea_uF;   // even part of the axis pairs
    R ed_sa, ed_sd, ed_r, ed_u2, ed_uF;   // even part of the diagonal pairs
    R pi_m, pi_F;                         // rows 10 and 12: moment and force
    R o_s, o_F;                           // odd part of the axis pairs
    R a_s, a_F, a_m;                      // odd part of the diagonal pairs
    R w_tr, c_tau;                        // tau_e - tau0 = c_tau sqrt(w), see collide;
                                          // kRescaled: w_tr is its square root
    R c3;        // 3 C (linear form) or 3 C^2; tau_e = tau0 + c3 |S|
    R a_e;       // s_e / (38 rho0): coefficient of m1_neq in S_aa (eq. yu_strain);
                 // 0 in the self-consistent mode
    R b9;        // s_9 / (2 rho0): coefficient of m9_neq in S_xx; s_9 = 1/tau0
                 // (explicit mode) or 1 (self-consistent mode: |S| = |S_1| / tau_e)
};

// The fixed relaxation rates.
struct Rates {
    double s_e, s_eps, s_q, s_pi, s_m;
};

// Result of the macroscopic / closure half of the collision.
template <typename R>
struct CellMacro {
    R drho;    // rho - rho0 (exact moment sum, kept for FP64 mass reductions)
    R rho, ux, uy, uz;
    R tau_t;   // tau_e - tau0 = 3 C Delta^2 |S| (or 3 C^2 Delta^2 |S|)
    R snorm2;  // |S|^2 = 2 S:S of the strain that sets tau_e (diagnostics only)
};

// The coefficients of collide from the rates and what k holds.  Every row of
// eq. mrt_les_guo is m* = (1 - s) m + s m_eq + (1 - s/2) F_m, a linear form of the
// pair sums and differences, the momentum, rho u u and u F; the rows with fixed
// rates are folded here into one coefficient per input and output.
// scale: the storage scale, in whose units collide's kScaled works.
inline void fill_collide_coefficients(CollideConst<double>& k, const Rates& rates,
                                      double scale = 1.0) {
    const double ge = 1.0 - 0.5 * rates.s_e, geps = 1.0 - 0.5 * rates.s_eps;
    // t1 = m1*/2394, t2 = m2*/252 as forms of (sa, sd, r, rho u^2, u.F), with
    // m1 = -11 sa + 8 sd - 30 r, m2 = -4 sa + sd + 12 r, t0 = (sa + sd + r)/19
    const double t0 = 1.0 / 19.0;
    const double t1[5] = {-11.0 / 2394.0, (8.0 - 19.0 * rates.s_e) / 2394.0,
                          (-30.0 + 19.0 * rates.s_e) / 2394.0, 19.0 * rates.s_e / 2394.0,
                          38.0 * ge / 2394.0};
    const double e2 = (1.0 - rates.s_eps) / 252.0;
    const double t2[5] = {-4.0 * e2, e2, 12.0 * e2, -475.0 / 63.0 * rates.s_eps / 252.0,
                          -11.0 * geps / 252.0};
    double* ea[5] = {&k.ea_sa, &k.ea_sd, &k.ea_r, &k.ea_u2, &k.ea_uF};
    double* ed[5] = {&k.ed_sa, &k.ed_sd, &k.ed_r, &k.ed_u2, &k.ed_uF};
    for (int i = 0; i < 5; ++i) {
        const double m = i < 3 ? t0 : 0.0;
        *ea[i] = m - 11.0 * t1[i] - 4.0 * t2[i];
        *ed[i] = m + 8.0 * t1[i] + t2[i];
    }
    k.pi_m = 1.0 - rates.s_pi;
    k.pi_F = -(1.0 - 0.5 * rates.s_pi);
    // odd rows: j* = rho u + F/2 and q* of rows 4, 6, 8 in terms of d0,
    // s0 = rho u_x - 3 d0 and F_x per axis; rows 16..18 as they are
    const double q = rates.s_q;
    k.o_s = q / 6.0;
    k.o_F = (2.0 - q) / 12.0;
    k.a_s = (3.0 - q) / 24.0;
    k.a_F = (1.0 + q) / 48.0;
    k.a_m = (1.0 - rates.s_m) / 8.0;
    // |S|^2 = 6 (a_e n1)^2 + b9^2 (3 n9^2 + 9 n11^2 + 36 (n13^2 + n14^2 + n15^2)),
    // n1 = 19 (sd - r - rho u^2)
    k.w_tr = 2.0 * (19.0 * k.a_e / k.b9) * (19.0 * k.a_e / k.b9);
    k.c_tau = k.c3 * k.b9 * 1.7320508075688772;
    // w is of the order of (rho0 scale)^2, its trace part of tau0^2 times that: out of
    // FP32 from rho0 = 2^64 or tau0 = 2^64 up, and at rho0 = 2^-43 a strain of 1e-6 is
    // lost.  Well before that it is formed of moments divided by a power of two.  (Where
    // w_tr ends at the type's largest value, tau0 is so large that the shear is kept whole
    // whatever w is, as long as it is a number.)
    int e, et;
    frexp(k.tau0, &et);
    frexp(k.rho0 * scale, &e);
    if (e > 32 || e < -16 || et > 20) {
        e += et > 0 ? et : 0;
        k.closure |= kRescaled | e * (1 << kScaleShift);
        k.w_tr = fmin(1.4142135623730951 * 19.0 * k.a_e / k.b9, DBL_MAX);
        k.c_tau = ldexp(k.c_tau, e) / scale;
    }
}

// One input's coefficients of the axis pairs (a) and the diagonal pairs (d) in FP32:
// of the values within 2 ulp of each, the two that also leave 6 a + 12 d nearest to
// its own value.  The rest population is what mass leaves after those 18, so that is
// its coefficient; rounded on their own, a and d left it up to 4e-8 off and its error
// after one step 1.3 times what rounding alone gives.
inline void round_even(double a, double d, float* fa, float* fd) {
    double best = INFINITY;
    for (int i = -2; i <= 2; ++i)
        for (int j = -2; j <= 2; ++j) {
            float x = (float)a, y = (float)d;
            for (int n = 0; n < abs(i); ++n) x = nextafterf(x, i < 0 ? -INFINITY : INFINITY);
            for (int n = 0; n < abs(j); ++n) y = nextafterf(y, j < 0 ? -INFINITY : INFINITY);
            const double ea = 6.0 * (x - a), ed = 12.0 * (y - d);
            const double cost = fabs(ea + ed) + 0.02 * (fabs(ea) + fabs(ed));
            if (cost < best) {
                best = cost;
                *fa = x;
                *fd = y;
            }
        }
}

// The same constants in FP32 arithmetic: each rounded once from its FP64 value, the
// even parts' coefficients in pairs.
inline CollideConst<float> round_constants(const CollideConst<double>& k) {
    CollideConst<float> f{};
    f.tau0 = (float)k.tau0; f.c3 = (float)k.c3; f.a_e = (float)k.a_e; f.b9 = (float)k.b9;
    f.rho0 = (float)k.rho0;
    f.tau0_sq = (float)k.tau0_sq; f.closure = k.closure;
    round_even(k.ea_sa, k.ed_sa, &f.ea_sa, &f.ed_sa);
    round_even(k.ea_sd, k.ed_sd, &f.ea_sd, &f.ed_sd);
    round_even(k.ea_r, k.ed_r, &f.ea_r, &f.ed_r);
    round_even(k.ea_u2, k.ed_u2, &f.ea_u2, &f.ed_u2);
    round_even(k.ea_uF, k.ed_uF, &f.ea_uF, &f.ed_uF);
    f.pi_m = (float)k.pi_m; f.pi_F = (float)k.pi_F;
    f.o_s = (float)k.o_s; f.o_F = (float)k.o_F;
    f.a_s = (float)k.a_s; f.a_F = (float)k.a_F; f.a_m = (float)k.a_m;
    f.w_tr = (float)fmin(k.w_tr, FLT_MAX); f.c_tau = (float)k.c_tau;
    return f;
}

// Macroscopic quantities and tau_e of one cell (diagnostics).  g: deviation
// populations, F: body force at the cell.
template <typename R>
__device__ __forceinline__ CellMacro<R> cell_macro(const R (&g)[19], R Fx, R Fy, R Fz,
                                                   const CollideConst<R>& k) {
    const R h = R(0.5);
    // pair sums (even rows) and differences (odd rows)
    const R p0 = g[0] + g[1], d0 = g[0] - g[1];
    const R p1 = g[2] + g[3], d1 = g[2] - g[3];
    const R p2 = g[4] + g[5], d2 = g[4] - g[5];
    const R p3 = g[6] + g[7], d3 = g[6] - g[7];
    const R p4 = g[8] + g[9], d4 = g[8] - g[9];
    const R p5 = g[10] + g[11], d5 = g[10] - g[11];
    const R p6 = g[12] + g[13], d6 = g[12] - g[13];
    const R p7 = g[14] + g[15], d7 = g[14] - g[15];
    const R p8 = g[16] + g[17], d8 = g[16] - g[17];
    const R r = g[18];

    // m = M g (eq. moment-matrix), deviation form
    const R sa = p0 + p1 + p2;                 // axis pairs
    const R sd = (p3 + p4) + (p5 + p6) + (p7 + p8);  // diagonal pairs
    const R m0 = sa + sd + r;                  // delta rho
    const R m1 = R(-11) * sa + R(8) * sd - R(30) * r;
    const R jx = d0 + d3 + d4 + d7 + d8;
    const R jy = d1 + d3 - d4 + d5 + d6;
    const R jz = d2 + d5 - d6 + d7 - d8;
    const R v9 = (p3 + p4) + (p7 + p8) - R(2) * (p5 + p6);
    const R m9 = R(2) * p0 - p1 - p2 + v9;
    const R v11 = (p3 + p4) - (p7 + p8);
    const R m11 = p1 - p2 + v11;
    const R m13 = p3 - p4;
    const R m14 = p5 - p6;
    const R m15 = p7 - p8;

    // eq. guo_velocity: rho u = sum f c + F/2
    const R rho = k.rho0 + m0;
    const R inv_rho = fast_rcp(rho);
    const R rux = jx + h * Fx, ruy = jy + h * Fy, ruz = jz + h * Fz;
    const R ux = rux * inv_rho, uy = ruy * inv_rho, uz = ruz * inv_rho;
    const R xx = rux * ux, yy = ruy * uy, zz = ruz * uz;   // rho u_a u_a
    const R ru2 = xx + yy + zz;

    // eq. meq_fm: the non-equilibrium parts the strain needs
    const R n1 = m1 - (R(-11) * m0 + R(19) * ru2);
    const R n9 = m9 - (R(2) * xx - yy - zz);
    const R n11 = m11 - (yy - zz);
    const R n13 = m13 - rux * uy;
    const R n14 = m14 - ruy * uz;
    const R n15 = m15 - rux * uz;

    // eq. yu_strain with s_1 = s_e, s_9 = 1/tau0 (explicit mode) or without the
    // s_1 term and s_9 = 1 (self-consistent mode, rescaled below); eq. strain_norm
    const R tr = k.a_e * n1;
    const R Sxx = -tr - k.b9 * n9;
    const R Syy = -tr + h * k.b9 * (n9 - R(3) * n11);
    const R Szz = -tr + h * k.b9 * (n9 + R(3) * n11);
    const R q = R(-3) * k.b9;
    const R Sxy = q * n13, Syz = q * n14, Sxz = q * n15;
    const R S2 = R(2) * (Sxx * Sxx + Syy * Syy + Szz * Szz) +
                 R(4) * (Sxy * Sxy + Sxz * Sxz + Syz * Syz);
    // eq. les_viscosity: tau_e = 1/2 + 3 (nu0 + C Delta^2 |S|) = tau0 + 3 C |S|
    R tau_t = k.c3 * fast_sqrt(S2);
    if (k.closure & kSelfConsistent) {
        // (the empty asm keeps this a uniform branch instead of computing it
        // always and selecting, so the default mode pays nothing for it)
        asm volatile("");
        // |S| = X / tau_e with X = |S_1| (computed above with s_9 = 1, no m1
        // term): tau_e^2 - tau0 tau_e - c3 X = 0.  Its positive root, as the
        // increment over tau0 without cancellation:
        // tau_e - tau0 = 2 c3 X / (tau0 + sqrt(tau0^2 + 4 c3 X)).
        tau_t = R(2) * tau_t * fast_rcp(k.tau0 + fast_sqrt(k.tau0_sq + R(4) * tau_t));
    }
    const R tau_e = k.tau0 + tau_t;
    // |S|^2: S2 itself, or (|S_1| / tau_e)^2 in the self-consistent mode
    const R snorm2 = (k.closure & kSelfConsistent) ? S2 * fast_rcp(tau_e * tau_e) : S2;
    return CellMacro<R>{m0, rho, ux, uy, uz, tau_t, snorm2};
}

__device__ __forceinline__ float mad(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double mad(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float scale2(float a, int e) { return __builtin_ldexpf(a, e); }
__device__ __forceinline__ double scale2(double a, int e) { return __builtin_ldexp(a, e); }

// Collide one cell in place (eq. mrt_les_guo).  g: deviation populations
// (pre-collision in, post-collision out).  F: body force at the cell.
//
// The step kernels are bound by the cache lines they move, but the instructions of the
// collision add to that where loads and stores are waited for (the VALUs are busy 23-29 %
// of the time in the one-step FP32 kernels, 39-44 % in the two-step one and 51-64 % with
// 16-bit storage), so the moments are never formed one by one: rows with a fixed rate are
// linear forms whose coefficients the host folds
// (fill_collide_coefficients), and only the five shear rows, whose rate differs
// per cell, are relaxed as moments.  With A = p3 + p4, B = p5 + p6, C = p7 + p8:
//   axis pairs, even:     ea +- ..., ea = forms of (sa, sd, r, rho u^2, u.F)
//   diagonal pairs, even: ed +- ...
//   rows 9 / 10:  m9 = a + b, m10 = b - 2 a,  a = 3 p0 - sa, b = sd - 3 B
//   rows 11 / 12: m11 = c + d, m12 = d - 2 c, c = p1 - p2,   d = A - C
//   odd parts:    o0 and ax, forms of d0, s = rho u_x - 3 d0 and F_x per axis;
//                 sums and differences of ax +- a_m m16, ay +- a_m m17, az +- a_m m18
// and |S|^2 needs n1 = 19 (sd - r - rho u^2), n9, n11, n13..15 squared only.  205
// floating-point instructions as compiled, where the row-by-row form took 268.
// Rounding: the populations are of order u, what changes in a step is much less, so
// the odd parts start from the old ones (d0/2 and d0/4, exact) and add terms that are
// zero in equilibrium: s, m16..18.  Momentum, 2 o0 + 8 ax = rho u_x + (2 o_s + 8 a_s - 1) s
// + ..., then keeps its rho u_x whatever the rates round to, and mass is kept by the rest
// population, which is what it leaves after the others.  Against 64 bits, 16 steps at
// 48^3: axis, diagonal and rest populations 1.2e-7, 1.6e-7, 4.5e-7 off in FP32 (the
// row-by-row form 2.9e-7, 3.1e-7, 7.1e-7), 2.2e-16, 3.0e-16, 8.3e-16 in FP64 (8.0e-16,
// 8.5e-16, 1.7e-15).
// Every product-sum is an explicit fused multiply-add and contraction is off, so
// all kernels that inline this give the same bits.
//
// kScaled: g and F come in units of 1/sigma (sigma g, sigma F, with sigma = 1/is
// a power of two: the 16-bit storage scale) and g leaves in the same units, so
// the storage codec needs no multiplications.  Every intermediate is then exactly
// sigma times its unscaled value (power-of-two scaling commutes with rounding);
// the places that need unscaled values (rho, 1/rho, tau_e) apply is, so the result
// equals sigma times the unscaled collision's, bit for bit.
template <typename R, bool kScaled = false>
__device__ __forceinline__ void collide(R (&g)[19], R Fx, R Fy, R Fz, const CollideConst<R>& k,
                                        R is = R(1)) {
#pragma clang fp contract(off)
    const R p0 = g[0] + g[1], d0 = g[0] - g[1];
    const R p1 = g[2] + g[3], d1 = g[2] - g[3];
    const R p2 = g[4] + g[5], d2 = g[4] - g[5];
    const R p3 = g[6] + g[7], d3 = g[6] - g[7];
    const R p4 = g[8] + g[9], d4 = g[8] - g[9];
    const R p5 = g[10] + g[11], d5 = g[10] - g[11];
    const R p6 = g[12] + g[13], d6 = g[12] - g[13];
    const R p7 = g[14] + g[15], d7 = g[14] - g[15];
    const R p8 = g[16] + g[17], d8 = g[16] - g[17];
    const R r = g[18];
    const R A = p3 + p4, B = p5 + p6, C = p7 + p8;
    const R sa = p0 + (p1 + p2), sd = B + (A + C);
    const R m0 = r + (sa + sd);                  // delta rho

    // eq. guo_velocity: rho u = sum f c + F/2 (rux.. and the products below carry
    // the scale of g; u itself is unscaled)
    const R rux = mad(R(0.5), Fx, d0 + ((d3 + d4) + (d7 + d8)));
    const R ruy = mad(R(0.5), Fy, d1 + ((d3 - d4) + (d5 + d6)));
    const R ruz = mad(R(0.5), Fz, d2 + ((d5 - d6) + (d7 - d8)));
    const R rho = kScaled ? mad(m0, is, k.rho0) : k.rho0 + m0;
    const R inv_rho = kScaled ? fast_rcp(rho) * is : fast_rcp(rho);
    const R ux = rux * inv_rho, uy = ruy * inv_rho, uz = ruz * inv_rho;
    const R xx = rux * ux, zz = ruz * uz;      // rho u_a u_a
    const R yz = mad(ruy, uy, zz), y_z = mad(ruy, uy, -zz);
    const R ru2 = xx + yz;
    const R XF = ux * Fx, ZF = uz * Fz;        // u_a F_a
    const R YZ = mad(uy, Fy, ZF), Y_Z = mad(uy, Fy, -ZF);
    const R uF = XF + YZ;
    const R PF = mad(R(2), XF, -YZ);           // 2 u_x F_x - u_y F_y - u_z F_z
    const R Fxy = mad(ux, Fy, uy * Fx), Fyz = mad(uy, Fz, uz * Fy), Fxz = mad(ux, Fz, uz * Fx);

    // shear rows and the trace: moments and their non-equilibrium parts (eq. meq_fm)
    const R a = mad(R(3), p0, -sa), b = mad(R(-3), B, sd);
    const R c = p1 - p2, d = A - C;
    const R m9 = a + b, m11 = c + d, m13 = p3 - p4, m14 = p5 - p6, m15 = p7 - p8;
    const R n1 = sd - r - ru2;
    const R n9 = m9 - mad(R(2), xx, -yz), n11 = m11 - y_z;
    const R n13 = mad(-rux, uy, m13), n14 = mad(-ruy, uz, m14), n15 = mad(-rux, uz, m15);

    // eq. yu_strain, eq. strain_norm, eq. les_viscosity: tau_e = tau0 + c_tau sqrt(w)
    // (the empty asm keeps the two branches uniform ones instead of computing both sides
    // and selecting, so the usual lattice pays nothing for them)
    R trace = n1 * n1, w_tr = k.w_tr, c_tau = kScaled ? k.c_tau * is : k.c_tau;
    R shear = mad(R(12), mad(n13, n13, mad(n14, n14, n15 * n15)), mad(R(3), n11 * n11, n9 * n9));
    if (__builtin_expect((k.closure & kRescaled) != 0, 0)) {
        asm volatile("");
        const int e = -(k.closure >> kScaleShift);
        const R t1 = k.w_tr * scale2(n1, e), t9 = scale2(n9, e), t11 = scale2(n11, e);
        const R t13 = scale2(n13, e), t14 = scale2(n14, e), t15 = scale2(n15, e);
        trace = t1 * t1;
        w_tr = R(1);
        shear = mad(R(12), mad(t13, t13, mad(t14, t14, t15 * t15)), mad(R(3), t11 * t11, t9 * t9));
        c_tau = k.c_tau;
    }
    R tau_t = c_tau * fast_sqrt(mad(w_tr, trace, shear));
    if (k.closure & kSelfConsistent) {
        asm volatile("");
        // the positive root of tau_e^2 - tau0 tau_e - c3 |S_1| = 0 as its
        // increment over tau0, as in cell_macro
        tau_t = R(2) * tau_t * fast_rcp(k.tau0 + fast_sqrt(mad(R(4), tau_t, k.tau0_sq)));
    }
    const R s = -fast_rcp(k.tau0 + tau_t);     // -s_nu

    // relaxed shear rows m + F_m - s_nu (m - m_eq + F_m / 2), rows 10 and 12
    const R q9 = mad(s, n9 + PF, mad(R(2), PF, m9));
    const R q10 = mad(k.pi_F, PF, k.pi_m * mad(R(-2), a, b));
    const R q11 = mad(s, n11 + Y_Z, mad(R(2), Y_Z, m11));
    const R q12 = mad(k.pi_F, Y_Z, k.pi_m * mad(R(-2), c, d));
    const R q13 = mad(s, mad(R(0.5), Fxy, n13), m13 + Fxy);
    const R q14 = mad(s, mad(R(0.5), Fyz, n14), m14 + Fyz);
    const R q15 = mad(s, mad(R(0.5), Fxz, n15), m15 + Fxz);

    // g* = M^-1 m*: even part per pair
    const R ea = mad(k.ea_uF, uF, mad(k.ea_u2, ru2, mad(k.ea_r, r, mad(k.ea_sd, sd, k.ea_sa * sa))));
    const R ed = mad(k.ed_uF, uF, mad(k.ed_u2, ru2, mad(k.ed_r, r, mad(k.ed_sd, sd, k.ed_sa * sa))));
    const R D9 = q9 - q10, D11 = q11 - q12;
    const R Q9 = mad(R(2), q9, q10), Q11 = mad(R(2), q11, q12);
    const R e0 = mad(R(1.0 / 18.0), D9, ea), ey = mad(R(-1.0 / 36.0), D9, ea);
    const R e1 = mad(R(1.0 / 12.0), D11, ey), e2 = mad(R(-1.0 / 12.0), D11, ey);
    const R ex = mad(R(1.0 / 72.0), Q9, ed), eyz = mad(R(-1.0 / 36.0), Q9, ed);
    const R exy = mad(R(1.0 / 24.0), Q11, ex), exz = mad(R(-1.0 / 24.0), Q11, ex);
    const R e3 = mad(R(0.25), q13, exy), e4 = mad(R(-0.25), q13, exy);
    const R e5 = mad(R(0.25), q14, eyz), e6 = mad(R(-0.25), q14, eyz);
    const R e7 = mad(R(0.25), q15, exz), e8 = mad(R(-0.25), q15, exz);
    // odd part per pair
    const R sx = mad(R(-3), d0, rux), sy = mad(R(-3), d1, ruy), sz = mad(R(-3), d2, ruz);
    const R o0 = mad(R(0.5), d0, mad(k.o_F, Fx, k.o_s * sx));
    const R o1 = mad(R(0.5), d1, mad(k.o_F, Fy, k.o_s * sy));
    const R o2 = mad(R(0.5), d2, mad(k.o_F, Fz, k.o_s * sz));
    const R ax = mad(R(0.25), d0, mad(k.a_F, Fx, k.a_s * sx));
    const R ay = mad(R(0.25), d1, mad(k.a_F, Fy, k.a_s * sy));
    const R az = mad(R(0.25), d2, mad(k.a_F, Fz, k.a_s * sz));
    const R m16 = (d3 + d4) - (d7 + d8);
    const R m17 = (d5 + d6) - (d3 - d4);
    const R m18 = (d7 - d8) - (d5 - d6);
    const R xp = mad(k.a_m, m16, ax), xm = mad(-k.a_m, m16, ax);
    const R yp = mad(k.a_m, m17, ay), ym = mad(-k.a_m, m17, ay);
    const R zp = mad(k.a_m, m18, az), zm = mad(-k.a_m, m18, az);
    const R o3 = xp + ym, o4 = xp - ym;
    const R o5 = yp + zm, o6 = yp - zm;
    const R o7 = xm + zp, o8 = xm - zp;

    g[0] = e0 + o0;  g[1] = e0 - o0;
    g[2] = e1 + o1;  g[3] = e1 - o1;
    g[4] = e2 + o2;  g[5] = e2 - o2;
    g[6] = e3 + o3;  g[7] = e3 - o3;
    g[8] = e4 + o4;  g[9] = e4 - o4;
    g[10] = e5 + o5; g[11] = e5 - o5;
    g[12] = e6 + o6; g[13] = e6 - o6;
    g[14] = e7 + o7; g[15] = e7 - o7;
    g[16] = e8 + o8; g[17] = e8 - o8;
    g[18] = mad(R(-12), ed, mad(R(-6), ea, m0));   // mass: m0 = 6 ea + 12 ed + g18
}

}  // namespace lbm
