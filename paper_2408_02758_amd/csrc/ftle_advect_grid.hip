// Flow maps by RK4 advection in a velocity field sampled on a regular grid,
// the form simulation output comes in (the paper's inputs are flow maps
// precomputed from such data, Section 2.2): nodes origin + i spacing per
// axis (x fastest), slices at t_first + k t_step.  The velocity is
// multilinear in space (bilinear in 2D, trilinear in 3D) and linear in time;
// a point outside the grid's box (a time outside the slices) takes the value
// at the nearest point of the box (the nearest slice).  One particle per
// lane, the classical fourth-order Runge-Kutta method in float64 with the
// steps of the analytic flows (ftle_advect.hip).
//
// Read plainly, every evaluation gathers its cell's corner values in two
// slices (64 bytes per particle in 2D) lane by lane, and those gathers bound
// the kernel.  A particle stays in a cell for a step or more and between the
// same two slices for many, so each lane keeps its cell's corner values in
// registers and reads the field only when its cell or slice pair changes.
// What is left is instruction issue, split between the evaluations and the
// misses (with 64 lanes to a wave, some lane leaves its cell in about two of a
// step's four stages), and both are kept short:
//  - the test whether a lane is still in its cell is the computation of its
//    cell fraction: f = position / spacing - (origin / spacing + cell), one FMA
//    from a constant kept with the cell, and f in [0, 1) is one unsigned compare
//    of its upper word (which also sends NaN, -0 and positions outside the box
//    to the full search);
//  - the corner values are blended in time once per stage time, not per stage
//    (two of the four stages share one, and a step starts where the last ended),
//    and turned into the polynomial's coefficients there, so that a stage is
//    2^D - 1 FMAs per component;
//  - a miss searches and loads, no more: the corner values stay in the field's
//    own type until they are blended (fewer registers: 84 instead of 95 in 2D),
//    and its offsets are 32-bit unless the field is 4 GiB.
// 1024 x 512 particles, 1500 steps in a 513 x 257 x 61 field: 348 -> 233 vector
// instructions a step, 7.61 -> 6.38 ms (the loads of 2.1 misses a step, 17 cache
// lines each, keep L1 and L2 busy two thirds of that); in a 129 x 65 x 61 field
// 6.95 -> 4.91 ms; steady 513 x 257, 512 x 512 particles: 2.67 -> 2.00 ms; 3D
// 97 x 96 x 97 x 21, 306,720 particles, 500 steps: 4.06 -> 3.73 ms.
// Against the definition's weighted sum of corner values, this and the
// reciprocal spacings reorder the arithmetic at the level of a rounding.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <type_traits>

#include "ftle_internal.h"

namespace ftle {
namespace {

// The field's constants in the form the kernel uses them: reciprocal
// spacings (a multiply in place of a divide; the cell and fraction then
// differ from a divide's by at most a rounding, and the interpolant is
// continuous across cell faces) and strides in elements.
struct GridArgs {
    double inv[3], base[3], top[3];   // 1 / spacing; -origin / spacing; shape - 1
    int cmax[3];                       // the last cell: shape - 2 (shapes below 2^31)
    int64_t stride[3];                 // elements between nodes along x, y, z
    int64_t slice;                     // elements between slices
    double inv_t, base_t, t_top;       // 1 / t_step; -t_first / t_step; nt - 1
    int kmax;                          // nt - 2 (nt below 2^31)
};

// A lane's current cell and slice pair.  In a cell the multilinear
// interpolant of one component is the polynomial sum over corner sets m of
// b_m prod_{d in m} f_d in the cell fractions f.
template <int D, bool TWO, typename V>
struct CellCache {
    static constexpr int kCorners = 1 << D;
    int cell[D], k;
    double cb[D], kb, w;   // base - cell; base_t - k; the weight of slice k + 1 at the stage's time
    V v0[TWO ? D : 1][kCorners], v1[TWO ? D : 1][kCorners];   // corner values in slices k and k + 1
    double b[D][kCorners];                       // the polynomial at the stage's time
};

// f in [0, 1), by the upper word: negative numbers and NaN compare as large.
__device__ inline bool in_unit(double f)
{
    return (uint32_t)((unsigned long long)__double_as_longlong(f) >> 32) < 0x3ff00000u;
}

// u clamped to [0, top] (NaN to 0), its cell c (at most cmax; 0 <= u < 2^31, so
// truncation is the floor) and the fraction u - c.
__device__ inline double search(double u, double top, int cmax, int& c)
{
    u = fmin(fmax(u, 0.0), top);
    c = min((int)u, cmax);
    return u - (double)c;
}

// A cell's corner values (corner m = x bit | y bit << 1 [| z bit << 2]) into
// the polynomial's coefficients: along each axis, the upper corners' values
// less the lower ones'.
template <int D>
__device__ inline void corners_to_coefficients(double* a)
{
#pragma unroll
    for (int d = 0; d < D; ++d)
#pragma unroll
        for (int m = 0; m < (1 << D); ++m)
            if (m & (1 << d)) a[m] -= a[m ^ (1 << d)];
}

// The polynomial at the cached weight.
template <int D, typename V>
__device__ inline void blend(CellCache<D, true, V>& cc)
{
#pragma unroll
    for (int d = 0; d < D; ++d) {
#pragma unroll
        for (int m = 0; m < CellCache<D, true, V>::kCorners; ++m)
            cc.b[d][m] = __builtin_fma(cc.w, (double)cc.v1[d][m] - (double)cc.v0[d][m], (double)cc.v0[d][m]);
        corners_to_coefficients<D>(cc.b[d]);
    }
}

// The corner values of the cached cell: per cell row along x the two x
// neighbours' components, 2 D consecutive values of the field.
template <int D, bool TWO, bool WIDE, typename V>
__device__ inline void load_cell(const GridArgs& g, const V* __restrict__ vel, CellCache<D, TWO, V>& cc)
{
    constexpr int kCorners = CellCache<D, TWO, V>::kCorners;
    using Off = std::conditional_t<WIDE, uint64_t, uint32_t>;
    Off off = TWO ? (Off)cc.k * (Off)g.slice : Off(0);
#pragma unroll
    for (int d = 0; d < D; ++d) off += (Off)cc.cell[d] * (Off)g.stride[d];
    off *= (Off)sizeof(V);
    auto at = [&](int r, bool second, int e) {
        const V* row = vel + ((r & 1) ? g.stride[1] : 0) + ((D == 3 && (r & 2)) ? g.stride[2] : 0) +
                       (second ? g.slice : 0);   // uniform
        return reinterpret_cast<const V*>(reinterpret_cast<const unsigned char*>(row) + off)[e];
    };
    V a[kCorners / 2][2 * D], c[kCorners / 2][2 * D];
#pragma unroll
    for (int r = 0; r < kCorners / 2; ++r)
#pragma unroll
        for (int e = 0; e < 2 * D; ++e) {
            a[r][e] = at(r, false, e);
            if constexpr (TWO) c[r][e] = at(r, true, e);
        }
#pragma unroll
    for (int r = 0; r < kCorners / 2; ++r)
#pragma unroll
        for (int e = 0; e < 2 * D; ++e) {
            const int d = e % D, m = 2 * r + e / D;
            if constexpr (TWO) {
                cc.v0[d][m] = a[r][e];
                cc.v1[d][m] = c[r][e];
            } else {
                cc.b[d][m] = (double)a[r][e];
            }
        }
    if constexpr (!TWO)
#pragma unroll
        for (int d = 0; d < D; ++d) corners_to_coefficients<D>(cc.b[d]);
}

// The velocity at p; TIME: at the new stage time t, otherwise at the time of
// the last call.
template <int D, bool TWO, bool WIDE, bool TIME, typename V>
__device__ inline void grid_velocity(const GridArgs& g, const V* __restrict__ vel, const double* p, double t,
                                     CellCache<D, TWO, V>& cc, double* v)
{
    double f[D];
    bool in = true;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        f[d] = __builtin_fma(p[d], g.inv[d], cc.cb[d]);
        in &= in_unit(f[d]);
    }
    if constexpr (TWO && TIME) {
        cc.w = __builtin_fma(t, g.inv_t, cc.kb);
        in &= in_unit(cc.w);
    }
    if (!in) {
        bool load = false;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            int c;
            f[d] = search(__builtin_fma(p[d], g.inv[d], g.base[d]), g.top[d], g.cmax[d], c);
            load |= c != cc.cell[d];
            cc.cell[d] = c;
            cc.cb[d] = g.base[d] - (double)c;
        }
        if constexpr (TWO && TIME) {
            int k;
            cc.w = search(__builtin_fma(t, g.inv_t, g.base_t), g.t_top, g.kmax, k);
            load |= k != cc.k;
            cc.k = k;
            cc.kb = g.base_t - (double)k;
        }
        if (load) {
            load_cell<D, TWO, WIDE>(g, vel, cc);
            if constexpr (TWO && !TIME) blend<D>(cc);
        }
    }
    if constexpr (TWO && TIME) blend<D>(cc);
#pragma unroll
    for (int d = 0; d < D; ++d) {
        double a[CellCache<D, TWO, V>::kCorners / 2];   // the polynomial in f, the highest axis folded first
#pragma unroll
        for (int m = 0; m < CellCache<D, TWO, V>::kCorners / 2; ++m)
            a[m] = __builtin_fma(f[D - 1], cc.b[d][m | (1 << (D - 1))], cc.b[d][m]);
#pragma unroll
        for (int e = D - 2; e >= 0; --e)
#pragma unroll
            for (int m = 0; m < (1 << e); ++m) a[m] = __builtin_fma(f[e], a[m | (1 << e)], a[m]);
        v[d] = a[0];
    }
}

template <int D, bool TWO, bool WIDE, bool EACH, typename T, typename V>
__global__ void __launch_bounds__(256) advect_grid_kernel(GridArgs g, const V* __restrict__ vel, int64_t n,
                                                          const T* __restrict__ x0, const double* __restrict__ t0s,
                                                          const double* __restrict__ Ts, double t0, double Tall,
                                                          double dt, double h_all, double half_all, double sixth_all,
                                                          int ns_all, T* __restrict__ phi)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double p[D], q[D], v[D], acc[D];
#pragma unroll
    for (int d = 0; d < D; ++d) p[d] = (double)x0[i * D + d];
    double ti = t0, h = h_all, half = half_all, sixth = sixth_all;
    int ns = ns_all;
    if constexpr (EACH) {
        if (t0s) ti = t0s[i];
        const double Ti = Ts ? Ts[i] : Tall;
        const double steps = fmax(1.0, ceil(fabs(Ti) / dt - 1e-9));
        if (!(steps <= (double)kMaxAdvectSteps)) {   // also NaN and inf
#pragma unroll
            for (int d = 0; d < D; ++d) phi[i * D + d] = (T)NAN;
            return;
        }
        h = Ti / steps;
        half = 0.5 * h;
        sixth = h / 6.0;
        ns = (int)steps;
    }
    CellCache<D, TWO, V> cc;
    cc.k = -1;   // no cell read yet: the fractions are NaN
    cc.kb = NAN;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        cc.cell[d] = -1;
        cc.cb[d] = NAN;
    }
    double t = ti;
    grid_velocity<D, TWO, WIDE, true>(g, vel, p, t, cc, acc);
    for (int s = 1;; ++s) {
        // acc: the velocity at the step's start
#pragma unroll
        for (int d = 0; d < D; ++d) q[d] = __builtin_fma(half, acc[d], p[d]);
        grid_velocity<D, TWO, WIDE, true>(g, vel, q, t + half, cc, v);
#pragma unroll
        for (int d = 0; d < D; ++d) {
            q[d] = __builtin_fma(half, v[d], p[d]);
            acc[d] = __builtin_fma(2.0, v[d], acc[d]);
        }
        grid_velocity<D, TWO, WIDE, false>(g, vel, q, 0.0, cc, v);
#pragma unroll
        for (int d = 0; d < D; ++d) {
            q[d] = __builtin_fma(h, v[d], p[d]);
            acc[d] = __builtin_fma(2.0, v[d], acc[d]);
        }
        t = __builtin_fma((double)s, h, ti);
        grid_velocity<D, TWO, WIDE, true>(g, vel, q, t, cc, v);
#pragma unroll
        for (int d = 0; d < D; ++d) p[d] = __builtin_fma(sixth, acc[d] + v[d], p[d]);
        if (s == ns) break;
        grid_velocity<D, TWO, WIDE, false>(g, vel, p, 0.0, cc, acc);
    }
#pragma unroll
    for (int d = 0; d < D; ++d) phi[i * D + d] = (T)p[d];
}

template <int D, typename T, typename V>
hipError_t advect_grid_launch(const GridField& g, const void* vel, int64_t n, const void* x0, const double* t0s,
                              const double* Ts, double t0, double T_, double dt, void* phi, hipStream_t stream)
{
    GridArgs a{};
    int64_t stride = D;
    for (int d = 0; d < D; ++d) {
        a.inv[d] = 1.0 / g.spacing[d];
        a.base[d] = -(g.origin[d] * a.inv[d]);
        a.top[d] = (double)(g.shape[d] - 1);
        a.cmax[d] = (int)(g.shape[d] - 2);
        a.stride[d] = stride;
        stride *= g.shape[d];
    }
    a.slice = stride;
    const bool two = g.nt > 1;
    a.inv_t = two ? 1.0 / g.t_step : 0.0;
    a.base_t = two ? -(g.t_first * a.inv_t) : 0.0;
    a.t_top = (double)(g.nt - 1);
    a.kmax = (int)(g.nt - 2);
    // Workgroups of four waves spread the waves evenly over the SIMDs while all
    // of them are resident at once (registers: four to eight a SIMD in 2D, two
    // to four in 3D); with more, single-wave workgroups, so that a wave that
    // ends makes room for the next without waiting for three others (misses
    // make their times uneven).  2D, 8192 waves: 64 threads 6.40 ms, 256 7.30;
    // 2D steady, 4096 waves (all resident): 64 threads 2.25 ms, 256 2.00.
    const int64_t resident = 1024 * (two ? (D == 2 ? 4 : 2) : (D == 2 ? 8 : 4));
    const int threads = (n + 63) / 64 <= resident ? 256 : 64;
    const int64_t blocks = (n + threads - 1) / threads;
    // 32-bit byte offsets while the field is below 4 GiB (they leave the
    // address arithmetic of a miss to the scalar unit)
    const bool wide = (double)stride * (double)g.nt * sizeof(V) >= 4294967296.0;
    // one window for all particles (the host has checked its step count): its
    // steps come as arguments and stay in scalar registers
    const bool each = t0s || Ts;
    const double steps = each ? 1.0 : std::fmax(1.0, std::ceil(std::fabs(T_) / dt - 1e-9));
    const double h = T_ / steps;
    const auto launch = [&](auto two_, auto wide_, auto each_) {
        hipLaunchKernelGGL((advect_grid_kernel<D, decltype(two_)::value, decltype(wide_)::value,
                                               decltype(each_)::value, T, V>),
                           dim3((unsigned)blocks), dim3(threads), 0, stream, a, static_cast<const V*>(vel), n,
                           static_cast<const T*>(x0), t0s, Ts, t0, T_, dt, h, 0.5 * h, h / 6.0, (int)steps,
                           static_cast<T*>(phi));
    };
    const auto with_each = [&](auto two_, auto wide_) {
        each ? launch(two_, wide_, std::true_type{}) : launch(two_, wide_, std::false_type{});
    };
    const auto with_wide = [&](auto two_) {
        wide ? with_each(two_, std::true_type{}) : with_each(two_, std::false_type{});
    };
    two ? with_wide(std::true_type{}) : with_wide(std::false_type{});
    return hipGetLastError();
}

}  // namespace

hipError_t launch_advect_grid(int dim, const GridField& g, const void* vel, bool vel_f64, bool f64, int64_t n,
                              const void* x0, const double* t0s, const double* Ts, double t0, double T, double dt,
                              void* phi, hipStream_t stream)
{
    if (n == 0) return hipSuccess;
#define FTLE_GRID(D, TT, VV) advect_grid_launch<D, TT, VV>(g, vel, n, x0, t0s, Ts, t0, T, dt, phi, stream)
    if (dim == 2) {
        if (f64) return vel_f64 ? FTLE_GRID(2, double, double) : FTLE_GRID(2, double, float);
        return vel_f64 ? FTLE_GRID(2, float, double) : FTLE_GRID(2, float, float);
    }
    if (f64) return vel_f64 ? FTLE_GRID(3, double, double) : FTLE_GRID(3, double, float);
    return vel_f64 ? FTLE_GRID(3, float, double) : FTLE_GRID(3, float, float);
#undef FTLE_GRID
}

}  // namespace ftle
