// kt_adjoint_math.h -- the pieces of the discrete adjoint that are pure
// arithmetic: Hamilton's equations, the
// vector-Jacobian product of the RHS as a Hessian-vector product, one
// Dormand-Prince step as a map y -> y' with frozen step size and its
// vector-Jacobian product, and the disk observables with their derivatives.
// Host and device: the same templates serve a host-side self-check.
#pragma once

#include "kt_dual.h"
#include "kt_elem.h"

namespace kt {
namespace adj {

// What the field and its derivatives share at one state, from Carter's
// separated form: H = K / (2 Sigma), K = Delta p_r^2 + p_th^2 + T^2 - W^2/Delta,
// T = L/sin - aE sin, W = (r^2 + a^2)E - aL.  (s, c) are sin and cos of theta;
// 1/sin, 1/Sigma and 1/Delta come from one reciprocal of their product.
struct Parts {
    double Del, rho2, iS, iD, is, T, W, Wd, G, H2, hdK, Q, X;  // Wd = W/Delta, H2 = 2H
};

__host__ __device__ inline __attribute__((always_inline)) Parts parts_at(double M, double a, double E, double L,
                                                                         const double z[5], double s, double c) {
    const double r = z[0], pr = z[3], pth = z[4];
    Parts p;
    const double a2 = a * a, r2 = r * r;
    const double Sig = r2 + a2 * c * c;
    p.Del = r * (r - 2.0 * M) + a2;
    p.rho2 = r2 + a2;
    const double SD = Sig * p.Del;
    const double R = rcp(SD * s);
    const double iSD = s * R;
    p.is = SD * R;
    p.iS = p.Del * iSD;
    p.iD = Sig * iSD;
    p.T = L * p.is - a * E * s;
    p.W = p.rho2 * E - a * L;
    p.Wd = p.W * p.iD;
    p.G = pr * pr + p.Wd * p.Wd;
    p.H2 = (p.Del * pr * pr + pth * pth + p.T * p.T - p.W * p.Wd) * p.iS;
    p.hdK = (r - M) * p.G - 2.0 * r * E * p.Wd;      // (1/2) dK/dr
    p.Q = L * p.is * p.is + a * E;                   // dT/dtheta = -cos Q
    p.X = p.T * p.Q - a2 * s * p.H2;                 // dH/dtheta = -cos X / Sigma
    return p;
}

// Hamilton's equations: d/dlambda (r, th, phi, p_r, p_th).  Returns sin and
// cos of theta (the trace kernel's own sincos_theta), which the step VJP
// reuses.
__host__ __device__ inline __attribute__((always_inline)) void field(double M, double a, double E, double L,
                                                                     const double z[5], double f[5], double* sv,
                                                                     double* cv) {
    sincos_theta(z[1], sv, cv);
    const Parts p = parts_at(M, a, E, L, z, *sv, *cv);
    f[0] = p.Del * z[3] * p.iS;
    f[1] = z[4] * p.iS;
    f[2] = (p.T * p.is + a * p.Wd) * p.iS;
    f[3] = (z[0] * p.H2 - p.hdK) * p.iS;
    f[4] = *cv * p.X * p.iS;
}

// Parameter cotangents accumulated along a ray.
struct ParBar {
    double E, L, a;
};

// Vector-Jacobian product of the field at z: zbar += (df/dz)^T v and the
// parameter cotangents += (df/d(E, L, a))^T v.  The field is S grad H, so
// this is the Hessian-vector product of H along u = (-v_pr, -v_th, v_r, v_th,
// v_phi) in (r, th, p_r, p_th, L): the derivative along u of each component
// g = N / Sigma of grad H, (dN - N dSigma/Sigma) / Sigma.  (sv, cv) are sin
// and cos of theta.  PHI false: v_phi is zero (phi enters no component of the
// field, so a cotangent without it stays without it), and its terms drop out.
//
// Written out: the same product by dual numbers through grad H took ~140
// vector instructions per stage, this ~115, and holds fewer values at once.
template <bool PHI = true>
__host__ __device__ inline __attribute__((always_inline)) void field_vjp(double M, double a, double E, double L,
                                                                         const double z[5], double sv, double cv,
                                                                         const double v[5], double zbar[5],
                                                                         ParBar* pb) {
    const double r = z[0], pr = z[3], pth = z[4], s = sv, c = cv, a2 = a * a;
    const double dr = -v[3], dth = -v[4], dpr = v[0], dpth = v[1];
    const Parts p = parts_at(M, a, E, L, z, s, c);
    const double rM = r - M, ds = c * dth, dc = -s * dth;
    const double dS = 2.0 * (r * dr + a2 * c * dc) * p.iS;  // dSigma / Sigma
    const double dDel = 2.0 * rM * dr;
    double dT = -p.Q * ds;
    double dW = 2.0 * r * E * dr;
    if (PHI) {
        dT += p.is * v[2];
        dW -= a * v[2];
    }
    const double dWd = (dW - p.Wd * dDel) * p.iD;
    const double dG = 2.0 * (pr * dpr + p.Wd * dWd);
    double hdK = p.hdK * dr + p.Del * pr * dpr + pth * dpth + p.T * dT;  // (1/2) dK
    if (PHI) hdK += a * p.Wd * v[2];
    const double dH2 = 2.0 * hdK * p.iS - p.H2 * dS;
    const double dhdK = dr * p.G + rM * dG - 2.0 * E * (dr * p.Wd + r * dWd);
    // numerators N of grad H and their derivatives
    const double Nr = p.hdK - r * p.H2;
    zbar[0] += (dhdK - dr * p.H2 - r * dH2 - Nr * dS) * p.iS;
    const double Lis2 = L * p.is * p.is;
    double dQ = -2.0 * Lis2 * p.is * ds;
    if (PHI) dQ += p.is * p.is * v[2];
    const double dX = dT * p.Q + p.T * dQ - a2 * (ds * p.H2 + s * dH2);
    zbar[1] += (c * p.X * dS - dc * p.X - c * dX) * p.iS;
    const double Npr = p.Del * pr;
    zbar[3] += (dDel * pr + p.Del * dpr - Npr * dS) * p.iS;
    zbar[4] += (dpth - pth * dS) * p.iS;
    const double NL = p.T * p.is + a * p.Wd;
    pb->L += (dT * p.is - p.T * p.is * p.is * ds + a * dWd - NL * dS) * p.iS;
    const double sT = s * p.T, dsT = ds * p.T + s * dT;
    const double NE = a * sT + p.rho2 * p.Wd;
    pb->E += (NE * dS - a * dsT - 2.0 * r * dr * p.Wd - p.rho2 * dWd) * p.iS;
    const double Wa = 2.0 * a * E - L;  // dW/da
    const double Na = a * p.G - E * sT - p.Wd * Wa - a * c * c * p.H2;
    double dNa = a * dG - E * dsT - dWd * Wa - a * c * (2.0 * dc * p.H2 + c * dH2);
    if (PHI) dNa += p.Wd * v[2];
    pb->a += (dNa - Na * dS) * p.iS;
}

// Dormand & Prince (1980) RK5(4)7M: the rows and 5th-order weights of the
// step map (the seventh stage only serves the error estimate and FSAL).
__host__ __device__ constexpr double dp_a(int i, int j) {
    constexpr double t[6][5] = {{0, 0, 0, 0, 0},
                                {1.0 / 5, 0, 0, 0, 0},
                                {3.0 / 40, 9.0 / 40, 0, 0, 0},
                                {44.0 / 45, -56.0 / 15, 32.0 / 9, 0, 0},
                                {19372.0 / 6561, -25360.0 / 2187, 64448.0 / 6561, -212.0 / 729, 0},
                                {9017.0 / 3168, -355.0 / 33, 46732.0 / 5247, 49.0 / 176, -5103.0 / 18656}};
    return t[i][j];
}
__host__ __device__ constexpr double dp_b(int j) {
    constexpr double t[6] = {35.0 / 384, 0, 500.0 / 1113, 125.0 / 192, -2187.0 / 6784, 11.0 / 84};
    return t[j];
}

// Keeps a stage of the reverse pass to itself on the device: what parts_at
// gave in the forward pass is recomputed from the stage state instead of kept
// (13 values per stage), and the scheduler does not mix stages.  The kernel that
// sweeps (the trace kernel's STORE form) then takes 249 VGPRs, two waves per SIMD,
// without a spill; left to itself the step VJP alone took 358 with 194 moves to and
// from the other half of the register file, or 77 scratch accesses per step at two
// waves.
template <bool PHI>
__host__ __device__ inline __attribute__((always_inline)) void stage_fence(double Y[5]) {
#ifdef __HIP_DEVICE_COMPILE__
#pragma unroll
    for (int i = 0; i < 5; ++i)
        if (PHI || i != 2) asm volatile("" : "+v"(Y[i]));
    __builtin_amdgcn_sched_barrier(0);
#else
    (void)Y;
#endif
}

// Vector-Jacobian product of one step with frozen h: given ybar at the
// step's end, returns ybar at its start (in place) and accumulates the
// parameter cotangents.  The stage states are rebuilt from y (the step's
// end value itself is not needed, so the last stage's field is skipped).
// Every loop is unrolled so that the stage arrays stay in registers: with
// run-time indices they would live in scratch memory, at half the speed.
// PHI false: ybar[2] is zero and stays so (see field_vjp), y[2] is not read.
template <bool PHI = true>
__host__ __device__ inline __attribute__((always_inline)) void dp_step_vjp(double M, double a, double E, double L,
                                                                           const double y[5], double h,
                                                                           double ybar[5], ParBar* pb) {
    double Y[6][5], K[5][5], S[6], C[6];
#pragma unroll
    for (int j = 0; j < 6; ++j) {
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            if (!PHI && i == 2) continue;
            double acc = 0.0;
#pragma unroll
            for (int l = 0; l < j; ++l) acc += dp_a(j, l) * K[l][i];
            Y[j][i] = y[i] + h * acc;
        }
        if (j < 5)
            field(M, a, E, L, Y[j], K[j], &S[j], &C[j]);
        else
            sincos_theta(Y[j][1], &S[j], &C[j]);
    }
    double kb[6][5];
#pragma unroll
    for (int j = 0; j < 6; ++j)
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            if (!PHI && i == 2) continue;
            kb[j][i] = h * dp_b(j) * ybar[i];
        }
#pragma unroll
    for (int j = 5; j >= 0; --j) {
        stage_fence<PHI>(Y[j]);
        double Yb[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
        field_vjp<PHI>(M, a, E, L, Y[j], S[j], C[j], kb[j], Yb, pb);
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            if (!PHI && i == 2) continue;
            ybar[i] += Yb[i];
#pragma unroll
            for (int l = 0; l < j; ++l) kb[l][i] += h * dp_a(j, l) * Yb[i];
        }
    }
}

// Observed intensity of a disk hit at radius r for a ray with constants
// (E, L), spin a and inner edge r_in (Keplerian rotation, or constant l0),
// as a dual number in (r, E, L, a, r_in).
struct DiskModel {
    double M, r_out, emis_q, l0;
    int rotation, emis_model;
};

__host__ __device__ inline Dual<5> disk_intensity(const DiskModel& dm, double r_, double E_, double L_, double a_,
                                                  double rin_) {
    using D = Dual<5>;
    const D r = D::var(r_, 0), E = D::var(E_, 1), L = D::var(L_, 2), a = D::var(a_, 3), rin = D::var(rin_, 4);
    const double M = dm.M;
    const D ir = 1.0 / r;
    const D gtt = -(1.0 - 2.0 * M * ir);
    const D gtp = -2.0 * M * a * ir;
    const D gpp = r * r + a * a + 2.0 * M * a * a * ir;
    D Om;
    if (dm.rotation == 1) {
        Om = -(gtp + dm.l0 * gtt) / (gpp + dm.l0 * gtp);
    } else {
        const double sM = sqrt(M);
        Om = sM / (r * dsqrt(r) + a * sM);
    }
    const D norm = -gtt - 2.0 * Om * gtp - Om * Om * gpp;
    const D g = dsqrt(norm) / (E - Om * L);
    D em;
    if (dm.emis_model == 1) {
        const D mr = M * ir;
        em = mr * mr * (1.0 - dsqrt(rin * ir));
        const D sv = (dm.r_out - r) / (2.0 * M);
        if (sv.v < 1.0) em = em * sv * sv * (3.0 - 2.0 * sv);
    } else {
        const double e0 = pow(M / r_, dm.emis_q);
        em = D(e0);
        em.d[0] = -dm.emis_q * e0 / r_;
    }
    return g * g * g * em;
}

// The seeds: cotangents from the intensity at crossing radius r_c with the crossing-time
// correction; (dr_c, dth_c) are r' and theta' there.
__host__ __device__ inline void seed(const DiskModel& dm, double a, double r_in, double r_c, double dr_c,
                                     double dth_c, double E, double L, double w, double zb[5], ParBar* pb,
                                     double* gr) {
    const Dual<5> I = disk_intensity(dm, r_c, E, L, a, r_in);
    *pb = ParBar{w * I.d[1], w * I.d[2], w * I.d[3]};
    *gr = w * I.d[4];
    const double rbar = w * I.d[0];
    // r_c = r(lambda*) with theta(lambda*) = pi/2: dr_c = dr - (r' / theta') dtheta
    zb[0] = rbar;
    zb[1] = -rbar * dr_c / dth_c;
    zb[2] = zb[3] = zb[4] = 0.0;
}

}  // namespace adj
}  // namespace kt
