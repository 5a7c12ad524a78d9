// kt_elem.h -- the elementary functions the trace kernel shares with the
// adjoint: the reciprocal and sin/cos of the polar angle.  sincos_theta is
// plain arithmetic and compiles on the host as well; rcp has a device form
// (the hardware estimate, refined) and a host form (a division), chosen by
// the side that calls it.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>

namespace kt {

// 1/x from the hardware reciprocal estimate y (relative error e) refined by
// one third-order step y (1 + e + e^2), which cubes the error (below 1e-21
// from the estimate's ~5e-8): the result is within about an ulp.
__device__ __forceinline__ double rcp(double x) {
    const double y = __builtin_amdgcn_rcp(x);
    const double e = fma(-x, y, 1.0);
    return fma(y, fma(e, e, e), y);
}
__host__ inline double rcp(double x) { return 1.0 / x; }

// a b + k for a constant k, as the three-operand FMA.  Left to itself the
// compiler takes the two-operand form, whose addend is overwritten, and copies
// k into a vector register pair before each use.  In the 3-wave build k is a
// scalar operand (set up by the scalar unit, which has slots to spare there);
// elsewhere a vector register pair.
__host__ __device__ constexpr bool inline_constant(double k) {
    return k == 0.5 || k == -0.5 || k == 1.0 || k == -1.0 || k == 2.0 || k == -2.0 || k == 4.0 || k == -4.0;
}
__device__ __forceinline__ double fma_k(double a, double b, double k) {
    if (__builtin_constant_p(k) && inline_constant(k)) return fma(a, b, k);
    double r;
#if defined(KT_WAVES_PER_EU) && KT_WAVES_PER_EU == 3
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "s"(k));
#else
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(k));
#endif
    return r;
}
__host__ inline double fma_k(double a, double b, double k) { return fma(a, b, k); }

// How the polynomials below take a Horner step a b + k: HornerFma as written;
// or with their constants in registers that a loop around them keeps.  For
// that, HornerK holds the constants of a function with two chains (the
// constant addends in call order, and each chain's leading coefficient; the
// second chain starts at call SECOND), HornerRecord fills it by running the
// function once, and HornerUse runs the function on it.  The compiler's own
// loop-invariant code motion gives up on these constants once registers look
// short and sets them up again for every step: three instructions each, 4-6%
// of the time of a wave alone on its SIMD (512x512 lensing 3.40 -> 3.22 ms).
// FORCED: with the three-operand FMA above; not in the long chains of
// sincos_theta outside the 3-wave build, which the scheduler then no longer
// interleaves with other work.
template <bool FORCED>
struct HornerFma {
    __host__ __device__ double operator()(double a, double b, double k) const {
#if defined(KT_WAVES_PER_EU) && KT_WAVES_PER_EU == 3
        return fma_k(a, b, k);
#else
        if constexpr (FORCED) return fma_k(a, b, k);
        return __builtin_fma(a, b, k);
#endif
    }
};
template <int CALLS, int SECOND>
struct HornerK {
    double k[CALLS], lead[2];
};
template <int CALLS, int SECOND>
struct HornerRecord {
    HornerK<CALLS, SECOND>* to;
    int n = 0;
    __device__ __forceinline__ double operator()(double a, double, double k) {
        if (n == 0) to->lead[0] = a;
        if (n == SECOND) to->lead[1] = a;
        to->k[n++] = k;
        return k;
    }
};
template <bool FORCED, int CALLS, int SECOND>
struct HornerUse {
    const HornerK<CALLS, SECOND>* from;
    int n = 0;
    __device__ __forceinline__ double operator()(double a, double b, double k) {
        const double x = n == 0 ? from->lead[0] : n == SECOND ? from->lead[1] : a;
        const double kept = from->k[n++];
        return HornerFma<FORCED>{}(x, b, inline_constant(k) ? k : kept);
    }
};
// Puts the constants into registers for good: the asm makes them opaque.
template <int CALLS, int SECOND>
__device__ __forceinline__ void pin(HornerK<CALLS, SECOND>* h) {
#pragma unroll
    for (int i = 0; i < 2; ++i) asm volatile("" : "+v"(h->lead[i]));
#pragma unroll
    for (int i = 0; i < CALLS; ++i) {
        if (inline_constant(h->k[i])) continue;
#if defined(KT_WAVES_PER_EU) && KT_WAVES_PER_EU == 3
        asm volatile("" : "+s"(h->k[i]));
#else
        asm volatile("" : "+v"(h->k[i]));
#endif
    }
}

// sin and cos of the polar angle theta.  theta is folded to t in [-pi, pi]
// by t = theta - 2 pi rint(theta / 2 pi) (t = theta exactly on [0, pi), the
// range of every ray that does not pass over the polar axis); then with
// u = |t| - pi/2 in [-pi/2, pi/2]: sin theta = copysign(cos u, t) and
// cos theta = -sin u.  cos u = 1 - x C(x) and sin u = u - u x S(x), x = u^2,
// with minimax polynomials C and S of degree 7 for |u| <= pi/2 (coefficients
// from minimax_coefs.py, the constant term of C held at 1/2).  With the
// coefficients rounded to double the absolute error stays below 1.4e-17 for
// cos u and 4.1e-17 for sin u, under a third of an ulp of 1; Taylor's series
// needs two more terms each for the same.  No quadrant selects.
template <class FMA = HornerFma<false>>
__host__ __device__ inline __attribute__((always_inline)) void sincos_theta(double th, double* s_out, double* c_out,
                                                                           FMA fma = FMA{}) {
    constexpr double INV_TWO_PI = 0.15915494309189533577;
    constexpr double TWO_PI_HI = 6.2831853071795862320e+00;  // 2 pi rounded to double
    constexpr double TWO_PI_LO = 2.4492935982947064e-16;     // 2 pi - TWO_PI_HI
    constexpr double PIO2_HI = 1.5707963267948965580e+00;
    constexpr double PIO2_LO = 6.1232339957367658e-17;
    const double n = __builtin_rint(th * INV_TWO_PI);
    double t = __builtin_fma(-n, TWO_PI_HI, th);
    t = __builtin_fma(-n, TWO_PI_LO, t);
    const double u = (fabs(t) - PIO2_HI) - PIO2_LO;
    const double u2 = u * u;
    double pc = 4.616135051438568e-14;
    pc = fma(pc, u2, -1.1463635437491283e-11);
    pc = fma(pc, u2, 2.0876592592498227e-09);
    pc = fma(pc, u2, -2.755731706851054e-07);
    pc = fma(pc, u2, 2.48015872857839e-05);
    pc = fma(pc, u2, -0.001388888888883005);
    pc = fma(pc, u2, 0.04166666666666583);
    pc = fma(pc, u2, -0.5);
    *s_out = __builtin_copysign(fma(pc, u2, 1.0), t);  // sin theta = +-cos u
    double ps = -2.7184963661503298e-15;
    ps = fma(ps, u2, 7.642712927256417e-13);
    ps = fma(ps, u2, -1.605892783643712e-10);
    ps = fma(ps, u2, 2.5052106606636936e-08);
    ps = fma(ps, u2, -2.755731920778693e-06);
    ps = fma(ps, u2, 0.00019841269841185962);
    ps = fma(ps, u2, -0.008333333333333115);
    ps = fma(ps, u2, 0.16666666666666666);
    *c_out = __builtin_fma(ps * u2, u, -u);  // cos theta = -sin u
}

}  // namespace kt
