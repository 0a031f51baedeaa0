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

// Velocity at p, with w the double gyre's time factor sin(omega t) at the
// stage's time (the steady ABC flow ignores it).
template <int KIND>
__device__ inline void flow_velocity(const FlowParams& pr, const double* p, double w, double* v)
{
    constexpr double kPi = 3.14159265358979323846;
    if constexpr (KIND == 0) {
        double cy, sy, sf, cf;
        const double a = pr.b * w, b = 1.0 - 2.0 * pr.b * w;
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
// The bounded path.  Particles whose whole path stays below kReach (bounded
// once, before the first step, from x0, T and the largest velocity) take
// steps with the sines and cosines written out below; the others (huge or
// non-finite coordinates and parameters) take general_steps.
//
// A step is float64 instruction issue and nothing else, so the work per stage
// decides.  The library's sincospi and sincos reduce to an eighth of a period
// and evaluate both functions of each argument, with the swaps and signs of
// eight octants.  Here:
//  - the double gyre's products of a sine and a cosine are two sines,
//      2 sin(pi f) cos(pi y) = sin(pi (f + y)) + sin(pi (f - y)),
//      2 cos(pi f) sin(pi y) = sin(pi (f + y)) - sin(pi (f - y)),
//    so a stage evaluates two odd polynomials on half a period instead of
//    four on an eighth.  y is first reduced to y - rint(y) (exact), so that the
//    sums carry no larger rounding than f itself and a particle on a wall (y an
//    integer) gets a normal velocity of exactly zero;
//  - the ABC flow's six values come from three reductions to half a period
//    (argument - k pi, pi in two parts), one sine and one cosine polynomial each
//    with the sign (-1)^k, no octant selects;
//  - the scale factors of the velocity are folded into the steps' h and h/6.
// The polynomials are Chebyshev economisations of the Taylor series with nine
// terms (gen_sincos_poly.py; dropped terms below 4e-18), so a velocity is as
// exact as the library's forms make it: about one rounding of the argument and
// one of the result, far below the rounding of the position, which a step
// makes once (80-bit reference, 4000 particles: rms error 1.4e-15 against
// 1.6e-15 over T = 5, 5.9e-14 against 5.8e-14 over T = 15).
// Vector instructions per step: double gyre 188 (library forms 435), ABC 359
// (778), all issued back to back (4.2 cycles each).  1024 x 512 particles, 1500
// double-gyre steps, float32: 3.94 ms (8.87); 81 x 67 x 59 particles, 500 ABC
// steps, float64: 1.56 ms (3.54).
// ---------------------------------------------------------------------------
constexpr double kReach = 1073741824.0;   // 2^30: periods fit the 32-bit parity below

// v, negated when the parity's lowest bit is set
__device__ inline double flip_sign(double v, uint32_t parity)
{
    return __longlong_as_double(__double_as_longlong(v) ^ (long long)((unsigned long long)(parity << 31) << 32));
}

// sin(pi (c - rint(c))) (-1)^(rint(c) + parity)
__device__ inline double sin_pi(double c, uint32_t parity)
{
#pragma clang fp contract(off)
    const double k = rint(c);
    const double r = c - k, z = r * r;
    double s = 7.697847275590284e-07;
    s = __builtin_fma(s, z, -2.1903499125519212e-05);
    s = __builtin_fma(s, z, 0.00046629981702308817);
    s = __builtin_fma(s, z, -0.007370430506093225);
    s = __builtin_fma(s, z, 0.08214588657312355);
    s = __builtin_fma(s, z, -0.599264529318946);
    s = __builtin_fma(s, z, 2.5501640398773007);
    s = __builtin_fma(s, z, -5.167712780049969);
    s = __builtin_fma(s, z, 3.141592653589793);
    return flip_sign(r, (uint32_t)(int)k + parity) * s;
}

__device__ inline void sin_cos(double x, double& sn, double& cs)
{
    const double k = rint(x * 0.3183098861837907);
    double r = __builtin_fma(k, -3.141592653589793, x);
    r = __builtin_fma(k, -1.2246467991473532e-16, r);
    const double z = r * r;
    const uint32_t parity = (uint32_t)(int)k;
    double s = 2.7215821926997076e-15;
    s = __builtin_fma(s, z, -7.643027273612204e-13);
    s = __builtin_fma(s, z, 1.6058940907182887e-10);
    s = __builtin_fma(s, z, -2.5052106891168703e-08);
    s = __builtin_fma(s, z, 2.755731921123654e-06);
    s = __builtin_fma(s, z, -0.0001984126984120872);
    s = __builtin_fma(s, z, 0.008333333333333186);
    s = __builtin_fma(s, z, -0.16666666666666666);
    double c = 4.608992189914223e-14;
    c = __builtin_fma(c, z, -1.1462903400770852e-11);
    c = __builtin_fma(c, z, 2.087656190004232e-09);
    c = __builtin_fma(c, z, -2.755731639228085e-07);
    c = __builtin_fma(c, z, 2.4801587277429444e-05);
    c = __builtin_fma(c, z, -0.0013888888888773081);
    c = __builtin_fma(c, z, 0.04166666666666388);
    c = __builtin_fma(c, z, -0.4999999999999997);
    c = __builtin_fma(c, z, 1.0);
    const double rs = flip_sign(r, parity);
    sn = __builtin_fma(rs * z, s, rs);
    cs = flip_sign(c, parity);
}

// Whether every argument of sin_pi / sin_cos on the path stays below kReach.
// A stage point lies within 2 |T| vmax of x0.  (False for NaN.)
template <int KIND>
__device__ inline bool bounded_path(const FlowParams& pr, const double* p, double T)
{
    constexpr double kPi = 3.14159265358979323846;
    if constexpr (KIND == 0) {
        const double va = 2.0 * fabs(T) * kPi * fabs(pr.a), e = fabs(pr.b);
        const double X = fabs(p[0]) + va;
        const double slope = 2.0 * e * X + 1.0 + 2.0 * e;   // >= |df/dx|, and slope * X >= |f|
        return X < kReach && slope * X < kReach && fabs(p[1]) + va * slope < kReach;
    } else {
        const double v = 2.0 * fabs(T) * (fabs(pr.a) + fabs(pr.b) + fabs(pr.c));
        return fabs(p[0]) + v < kReach && fabs(p[1]) + v < kReach && fabs(p[2]) + v < kReach;
    }
}

// The double gyre's velocity at p over (-pi A / 2, pi A / 2), with
// a = eps sin(omega t) at the stage's time.  (No contraction beyond the written
// FMAs: on a wall the two sines are the same number and have to cancel.)
__device__ inline void gyre_stage(const double* p, double a, double* v)
{
#pragma clang fp contract(off)
    const double g = __builtin_fma(a, p[0], __builtin_fma(a, -2.0, 1.0));   // f = g x, df/dx = g + a x
    const double ky = rint(p[1]), ry = p[1] - ky;
    const uint32_t parity = (uint32_t)(int)ky;
    const double sp = sin_pi(__builtin_fma(g, p[0], ry), parity);
    const double sm = sin_pi(__builtin_fma(g, p[0], -ry), parity);
    v[0] = sp + sm;
    v[1] = (sp - sm) * __builtin_fma(a, p[0], g);
}

// The four stages of a double-gyre step take its time factor sin(omega t) at
// t, t + h/2 (twice) and t + h.  eps (sin, cos)(omega t) advances by a
// rotation through omega h per step (the half step's value by one through
// omega h / 2) and is evaluated directly every kAnchor steps: a rotation with
// rounded coefficients moves the pair by a few units in the last place, so the
// drift stays below 10^-13, far under the RK4 truncation error, at two
// instructions per value instead of a sine.
constexpr int kAnchor = 32;

template <int KIND>
__device__ inline void bounded_steps(const FlowParams& pr, double* p, double ti, double h, int64_t ns)
{
    constexpr double kPi = 3.14159265358979323846;
    if constexpr (KIND == 0) {
        double rsh, rch, rsf, rcf;
        sincos(pr.c * (0.5 * h), &rsh, &rch);
        sincos(pr.c * h, &rsf, &rcf);
        const double full[2] = {-0.5 * kPi * pr.a * h, 0.5 * kPi * pr.a * h};
        const double half[2] = {0.5 * full[0], 0.5 * full[1]};
        const double sixth[2] = {full[0] / 6.0, full[1] / 6.0};
        for (int64_t s0 = 0; s0 < ns; s0 += kAnchor) {
            double a, ac;
            sincos(pr.c * (ti + (double)s0 * h), &a, &ac);
            a *= pr.b;
            ac *= pr.b;
            const int m = (int)min((int64_t)kAnchor, ns - s0);
            for (int j = 0; j < m; ++j) {
                const double ah = __builtin_fma(a, rch, ac * rsh);
                const double a1 = __builtin_fma(a, rcf, ac * rsf);
                ac = __builtin_fma(ac, rcf, -(a * rsf));
                // the stages' sum in velocity units, so that a step rounds the
                // position once
                double v[2], q[2], acc[2];
                gyre_stage(p, a, acc);
#pragma unroll
                for (int d = 0; d < 2; ++d) q[d] = __builtin_fma(half[d], acc[d], p[d]);
                gyre_stage(q, ah, v);
#pragma unroll
                for (int d = 0; d < 2; ++d) {
                    q[d] = __builtin_fma(half[d], v[d], p[d]);
                    acc[d] = __builtin_fma(2.0, v[d], acc[d]);
                }
                gyre_stage(q, ah, v);
#pragma unroll
                for (int d = 0; d < 2; ++d) {
                    q[d] = __builtin_fma(full[d], v[d], p[d]);
                    acc[d] = __builtin_fma(2.0, v[d], acc[d]);
                }
                gyre_stage(q, a1, v);
#pragma unroll
                for (int d = 0; d < 2; ++d) p[d] = __builtin_fma(sixth[d], acc[d] + v[d], p[d]);
                a = a1;
            }
        }
    } else {
        const double half = 0.5 * h, sixth = h / 6.0;
        auto stage = [&](const double* x, double* v) {
            double s[3], c[3];
#pragma unroll
            for (int d = 0; d < 3; ++d) sin_cos(x[d], s[d], c[d]);
            v[0] = __builtin_fma(pr.a, s[2], pr.c * c[1]);
            v[1] = __builtin_fma(pr.b, s[0], pr.a * c[2]);
            v[2] = __builtin_fma(pr.c, s[1], pr.b * c[0]);
        };
        for (int64_t s = 0; s < ns; ++s) {
            double v[3], q[3], acc[3];
            stage(p, acc);
#pragma unroll
            for (int d = 0; d < 3; ++d) q[d] = __builtin_fma(half, acc[d], p[d]);
            stage(q, v);
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                q[d] = __builtin_fma(half, v[d], p[d]);
                acc[d] = __builtin_fma(2.0, v[d], acc[d]);
            }
            stage(q, v);
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                q[d] = __builtin_fma(h, v[d], p[d]);
                acc[d] = __builtin_fma(2.0, v[d], acc[d]);
            }
            stage(q, v);
#pragma unroll
            for (int d = 0; d < 3; ++d) p[d] = __builtin_fma(sixth, acc[d] + v[d], p[d]);
        }
    }
}

// Any path, by the math library's sines and cosines.
template <int KIND>
__device__ inline void general_steps(const FlowParams& pr, double* p, double ti, double h, int64_t ns)
{
    constexpr int D = KIND == 0 ? 2 : 3;
    double q[D], k1[D], k2[D], k3[D], k4[D];
    for (int64_t s = 0; s < ns; ++s) {
        const double t = ti + (double)s * h;
        flow_velocity<KIND>(pr, p, KIND == 0 ? sin(pr.c * t) : 0.0, k1);
        const double wh = KIND == 0 ? sin(pr.c * (t + 0.5 * h)) : 0.0;
#pragma unroll
        for (int d = 0; d < D; ++d) q[d] = p[d] + 0.5 * h * k1[d];
        flow_velocity<KIND>(pr, q, wh, k2);
#pragma unroll
        for (int d = 0; d < D; ++d) q[d] = p[d] + 0.5 * h * k2[d];
        flow_velocity<KIND>(pr, q, wh, k3);
#pragma unroll
        for (int d = 0; d < D; ++d) q[d] = p[d] + h * k3[d];
        flow_velocity<KIND>(pr, q, KIND == 0 ? sin(pr.c * (t + h)) : 0.0, k4);
#pragma unroll
        for (int d = 0; d < D; ++d) p[d] += h / 6.0 * (k1[d] + 2.0 * k2[d] + 2.0 * k3[d] + k4[d]);
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
    if (bounded_path<KIND>(pr, p, Ti))
        bounded_steps<KIND>(pr, p, ti, h, ns);
    else
        general_steps<KIND>(pr, p, ti, h, ns);
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
