// Flow maps by advection on the GPU: the step before the FTLE path.  The
// paper's inputs are flow maps precomputed by an advection code (UVaFTLE,
// Section 2.2); this computes them for analytic velocity fields, one particle
// per lane, by the classical fourth-order Runge-Kutta method in float64.
//
// Flows (their definitions, not anyone's code):
//  - the double gyre of Shadden, Lekien and Marsden (Physica D 212, 2005):
//    stream function psi = A sin(pi f) sin(pi y), f = eps sin(omega t) x^2 +
//    (1 - 2 eps sin(omega t)) x, velocity (-dpsi/dy, dpsi/dx);
//  - the steady Arnold-Beltrami-Childress flow
//    (A sin z + C cos y, B sin x + A cos z, C sin y + B cos x).
//
// A particle takes max(1, ceil(|T|/dt - 1e-9)) steps of T/steps from t0; a
// particle whose duration is not finite or needs more than kMaxAdvectSteps
// steps gets NaN without stepping (the host rejects such a common T).
// The work is arithmetic on registers: one 2-3 value load and one store per
// particle.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "ftle_internal.h"

namespace ftle {
namespace {

struct FlowParams {
    double a, b, c;
};

// Velocity at p by the math library's sines and cosines, with a the double
// gyre's eps sin(omega t) at the stage's time (the steady ABC flow ignores it).
template <int KIND>
__device__ inline void flow_velocity(const FlowParams& pr, const double* p, double a, double* v)
{
    constexpr double kPi = 3.14159265358979323846;
    if constexpr (KIND == 0) {
        double cy, sy, sf, cf;
        const double b = 1.0 - 2.0 * a;
        const double f = (a * p[0] + b) * p[0];
        const double dfdx = 2.0 * a * p[0] + b;
        sincospi(p[1], &sy, &cy);
        sincospi(f, &sf, &cf);
        v[0] = -kPi * pr.a * sf * cy;
        v[1] = kPi * pr.a * cf * sy * dfdx;
    } else {
        double sx, cx, sy, cy, sz, cz;
        sincos(p[0], &sx, &cx);
        sincos(p[1], &sy, &cy);
        sincos(p[2], &sz, &cz);
        v[0] = pr.a * sz + pr.c * cy;
        v[1] = pr.b * sx + pr.a * cz;
        v[2] = pr.c * sy + pr.b * cx;
    }
}

// ---------------------------------------------------------------------------
// The bounded path.  Blocks of steps on which every argument stays below kReach
// (known from the position, their duration and the largest velocity) take the
// sines and cosines written out below; the others (huge or non-finite
// coordinates and parameters) take flow_velocity's.
//
// A step is float64 instruction issue and nothing else, so the work per stage
// decides.  The library's sincospi and sincos reduce to an eighth of a period
// and evaluate both functions of each argument, with the swaps and signs of
// eight octants.  Here:
//  - the double gyre's four factors are odd polynomials on half a period: the
//    sines of f - rint(f) and y - rint(y) (exact), the cosines of the distance
//    to their own zero, 1/2 - |.|, and one sign for both products.  Odd
//    polynomials keep a factor's relative exactness at its zero, so that a
//    particle next to a wall leaves it as it should and one on a wall (y an
//    integer, x = 0) has a normal velocity of exactly zero (two sines, of f + y
//    and f - y, would do for all four, but their sum and difference cancel
//    there: 4.09 ms where this takes 5.80, and 1e-16 absolute);
//  - the ABC flow's six values come from three reductions to a quarter of a
//    period, with the reduced argument's rounding carried along, so that its
//    sines and cosines are as exact as the library's (rms error 2.8e-17);
//  - the scale factors of the velocity are folded into the steps' h and h/6.
// The polynomials are Chebyshev economisations of the Taylor series
// (gen_sincos_poly.py; dropped terms below 2e-17 of a term that is itself at
// most 0.6).  Against binary128 a double-gyre velocity's rms error is 4.8e-17
// (5.5e-17 with the library's functions), 1.3e-16 of it next to a wall (1.6e-16);
// an ABC velocity's 9.8e-17 (9.7e-17).
// Vector instructions per step: double gyre 267 (library forms 435), ABC 506
// (778), issued back to back.  1024 x 512 particles, 1500 double-gyre steps,
// float32: 5.80 ms (8.86); 81 x 67 x 59 particles, 500 ABC steps, float64:
// 2.17 ms (3.53).
//
// The bound is taken per block: over a whole path it grows with the square of
// the duration and sent the double gyre to the library's forms from 7e4 time
// units on (1024 particles, 2e5 steps of 0.5: 245 ms by whole paths, 98 by
// blocks).
// ---------------------------------------------------------------------------
constexpr double kReach = 1073741824.0;   // 2^30: periods fit the 32-bit parity below

// v, negated when the parity's lowest bit is set
__device__ inline double flip_sign(double v, uint32_t parity)
{
    return __hiloint2double((int)((uint32_t)__double2hiint(v) ^ (parity << 31 & 0x80000000u)), __double2loint(v));
}

// sin(pi r) / pi, |r| <= 1/2
__device__ inline double half_sine(double r)
{
    const double z = r * r;
    double s = 2.45918692848767e-07;
    s = __builtin_fma(s, z, -6.972961128185442e-06);
    s = __builtin_fma(s, z, 0.00014842817836379502);
    s = __builtin_fma(s, z, -0.002346080963525959);
    s = __builtin_fma(s, z, 0.026147847813081743);
    s = __builtin_fma(s, z, -0.1907518241219414);
    s = __builtin_fma(s, z, 0.8117424252833519);
    s = __builtin_fma(s, z, -1.6449340668482264);
    return __builtin_fma(r * z, s, r);
}

// sin x and cos x: r = x - k pi / 2 with its rounding t (the first product's
// difference is exact), sine and cosine polynomials on |r| <= pi / 4 whose last
// sum alone rounds, swapped and signed by k's quadrant.
__device__ inline void sin_cos(double x, double& sn, double& cs)
{
#pragma clang fp contract(off)
    const double k = rint(x * 0.6366197723675814);
    const double r1 = __builtin_fma(k, -1.5707963267948966, x);
    const double r = __builtin_fma(k, -6.123233995736766e-17, r1);
    const double t = __builtin_fma(k, -6.123233995736766e-17, r1 - r);
    const double z = r * r;
    double s = 1.5918135932869774e-10;
    s = __builtin_fma(s, z, -2.5051131947374594e-08);
    s = __builtin_fma(s, z, 2.7557316103105014e-06);
    s = __builtin_fma(s, z, -0.0001984126983675979);
    s = __builtin_fma(s, z, 0.00833333333333095);
    s = __builtin_fma(s, z, -0.16666666666666666);
    s = r + __builtin_fma(r * z, s, t);
    double c = -1.1382636115964061e-11;
    c = __builtin_fma(c, z, 2.087614632531677e-09);
    c = __builtin_fma(c, z, -2.7557317272036996e-07);
    c = __builtin_fma(c, z, 2.4801587298766363e-05);
    c = __builtin_fma(c, z, -0.0013888888888887398);
    c = __builtin_fma(c, z, 0.041666666666666664);
    const double w = __builtin_fma(-0.5, z, 1.0);
    c = w + __builtin_fma(z * z, c, __builtin_fma(-r, t, __builtin_fma(-0.5, z, 1.0 - w)));
    const uint32_t q = (uint32_t)(int)k;
    sn = flip_sign(q & 1 ? c : s, q >> 1);
    cs = flip_sign(q & 1 ? -s : c, q >> 1);
}

// Whether every argument (and the double gyre's f and y together) stays below
// kReach on a path of duration T from p: a stage point lies within 2 |T| vmax of
// p.  (False for NaN.)
template <int KIND>
__device__ inline bool bounded_path(const FlowParams& pr, const double* p, double T)
{
    constexpr double kPi = 3.14159265358979323846;
    if constexpr (KIND == 0) {
        const double va = 2.0 * fabs(T) * kPi * fabs(pr.a), e = fabs(pr.b);
        const double X = fabs(p[0]) + va;
        const double slope = 2.0 * e * X + 1.0 + 2.0 * e;   // >= |df/dx|, and slope * X >= |f|
        return X < kReach && slope * X + fabs(p[1]) + va * slope < kReach;
    } else {
        const double v = 2.0 * fabs(T) * (fabs(pr.a) + fabs(pr.b) + fabs(pr.c));
        return fabs(p[0]) + v < kReach && fabs(p[1]) + v < kReach && fabs(p[2]) + v < kReach;
    }
}

// The double gyre's velocity at p over (-pi^3 A, pi^3 A), with
// a = eps sin(omega t) at the stage's time.
__device__ inline void gyre_stage(const double* p, double a, double* v)
{
#pragma clang fp contract(off)
    const double g = __builtin_fma(a, p[0], __builtin_fma(a, -2.0, 1.0));   // f = g x, df/dx = g + a x
    const double kf = rint(g * p[0]), rf = __builtin_fma(g, p[0], -kf);
    const double ky = rint(p[1]), ry = p[1] - ky;
    const uint32_t parity = (uint32_t)(int)(kf + ky);   // the sign of both products
    const double sf = half_sine(flip_sign(rf, parity)), cf = half_sine(0.5 - fabs(rf));
    const double sy = half_sine(flip_sign(ry, parity)), cy = half_sine(0.5 - fabs(ry));
    v[0] = sf * cy;
    v[1] = cf * sy * __builtin_fma(a, p[0], g);
}

// The velocity of a stage (BOUNDED double gyre: over its scale, which rk4_steps
// folds into h), with a = eps sin(omega t) at the stage's time.
template <int KIND, bool BOUNDED>
__device__ inline void stage(const FlowParams& pr, const double* p, double a, double* v)
{
    if constexpr (!BOUNDED) {
        flow_velocity<KIND>(pr, p, a, v);
    } else if constexpr (KIND == 0) {
        gyre_stage(p, a, v);
    } else {
        double s[3], c[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) sin_cos(p[d], s[d], c[d]);
        v[0] = __builtin_fma(pr.a, s[2], pr.c * c[1]);
        v[1] = __builtin_fma(pr.b, s[0], pr.a * c[2]);
        v[2] = __builtin_fma(pr.c, s[1], pr.b * c[0]);
    }
}

// The four stages of a double-gyre step take its time factor sin(omega t) at
// t, t + h/2 (twice) and t + h.  eps (sin, cos)(omega t) advances by a
// rotation through omega h per step (the half step's value by one through
// omega h / 2) and is evaluated directly every kAnchor steps: a rotation with
// rounded coefficients moves the pair by a few units in the last place, so the
// drift stays below 10^-13, far under the RK4 truncation error, at two
// instructions per value instead of a sine.
constexpr int kAnchor = 32;

struct Rotation {
    double sh, ch, sf, cf;   // sine and cosine of omega h / 2 and omega h
};

// m steps of h from p, with (a, ac) = eps (sin, cos)(omega t) at their start.
template <int KIND, bool BOUNDED>
__device__ inline void rk4_steps(const FlowParams& pr, double* p, double a, double ac, const Rotation& rot, double h,
                                 int m)
{
    constexpr int D = KIND == 0 ? 2 : 3;
    double full[D], half[D], sixth[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        constexpr double kPi3 = 31.00627668029982;   // pi^3 (to 1.4e-17 of it)
        full[d] = !BOUNDED || KIND == 1 ? h : (d == 0 ? -kPi3 : kPi3) * (pr.a * h);
        half[d] = 0.5 * full[d];
        sixth[d] = full[d] / 6.0;
    }
    for (int j = 0; j < m; ++j) {
        double ah = 0.0, a1 = 0.0;
        if constexpr (KIND == 0) {
            ah = __builtin_fma(a, rot.ch, ac * rot.sh);
            a1 = __builtin_fma(a, rot.cf, ac * rot.sf);
            ac = __builtin_fma(ac, rot.cf, -(a * rot.sf));
        }
        // the stages' sum in velocity units, so that a step rounds the position once
        double v[D], q[D], acc[D];
        stage<KIND, BOUNDED>(pr, p, a, acc);
#pragma unroll
        for (int d = 0; d < D; ++d) q[d] = __builtin_fma(half[d], acc[d], p[d]);
        stage<KIND, BOUNDED>(pr, q, ah, v);
#pragma unroll
        for (int d = 0; d < D; ++d) {
            q[d] = __builtin_fma(half[d], v[d], p[d]);
            acc[d] = __builtin_fma(2.0, v[d], acc[d]);
        }
        stage<KIND, BOUNDED>(pr, q, ah, v);
#pragma unroll
        for (int d = 0; d < D; ++d) {
            q[d] = __builtin_fma(full[d], v[d], p[d]);
            acc[d] = __builtin_fma(2.0, v[d], acc[d]);
        }
        stage<KIND, BOUNDED>(pr, q, a1, v);
#pragma unroll
        for (int d = 0; d < D; ++d) p[d] = __builtin_fma(sixth[d], acc[d] + v[d], p[d]);
        a = a1;
    }
}

template <int KIND, typename T>
__global__ void __launch_bounds__(256) advect_kernel(FlowParams pr, int64_t n, const T* __restrict__ x0,
                                                     const double* __restrict__ t0s, const double* __restrict__ Ts,
                                                     double t0, double Tall, double dt, T* __restrict__ phi)
{
    constexpr int D = KIND == 0 ? 2 : 3;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double p[D];
#pragma unroll
    for (int d = 0; d < D; ++d) p[d] = (double)x0[i * D + d];
    const double ti = t0s ? t0s[i] : t0;
    const double Ti = Ts ? Ts[i] : Tall;
    const double steps = fmax(1.0, ceil(fabs(Ti) / dt - 1e-9));
    if (!(steps <= (double)kMaxAdvectSteps)) {   // also NaN and inf
#pragma unroll
        for (int d = 0; d < D; ++d) phi[i * D + d] = (T)NAN;
        return;
    }
    const double h = Ti / steps;
    const int64_t ns = (int64_t)steps;
    Rotation rot{};
    if constexpr (KIND == 0) {
        sincos(pr.c * (0.5 * h), &rot.sh, &rot.ch);
        sincos(pr.c * h, &rot.sf, &rot.cf);
    }
    for (int64_t s = 0; s < ns; s += kAnchor) {
        const int m = (int)min((int64_t)kAnchor, ns - s);
        double a = 0.0, ac = 0.0;
        if constexpr (KIND == 0) {
            sincos(pr.c * (ti + (double)s * h), &a, &ac);
            a *= pr.b;
            ac *= pr.b;
        }
        if (bounded_path<KIND>(pr, p, m * h))
            rk4_steps<KIND, true>(pr, p, a, ac, rot, h, m);
        else
            rk4_steps<KIND, false>(pr, p, a, ac, rot, h, m);
    }
#pragma unroll
    for (int d = 0; d < D; ++d) phi[i * D + d] = (T)p[d];
}

template <int KIND, typename T>
hipError_t advect_launch(const FlowParams& pr, int64_t n, const void* x0, const double* t0s, const double* Ts,
                         double t0, double T_, double dt, void* phi, hipStream_t stream)
{
    const int64_t blocks = (n + 255) / 256;
    hipLaunchKernelGGL((advect_kernel<KIND, T>), dim3((unsigned)blocks), dim3(256), 0, stream, pr, n,
                       static_cast<const T*>(x0), t0s, Ts, t0, T_, dt, static_cast<T*>(phi));
    return hipGetLastError();
}

}  // namespace

hipError_t launch_advect(int kind, const double* params, bool f64, int64_t n, const void* x0, const double* t0s,
                         const double* Ts, double t0, double T, double dt, void* phi, hipStream_t stream)
{
    if (n == 0) return hipSuccess;
    const FlowParams pr{params[0], params[1], params[2]};
    if (kind == 0)
        return f64 ? advect_launch<0, double>(pr, n, x0, t0s, Ts, t0, T, dt, phi, stream)
                   : advect_launch<0, float>(pr, n, x0, t0s, Ts, t0, T, dt, phi, stream);
    return f64 ? advect_launch<1, double>(pr, n, x0, t0s, Ts, t0, T, dt, phi, stream)
               : advect_launch<1, float>(pr, n, x0, t0s, Ts, t0, T, dt, phi, stream);
}

}  // namespace ftle
