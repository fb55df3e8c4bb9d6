// Occupations, Fermi energy and electron density (Sec. 3.4).
//
// After the Rayleigh-Ritz step the Fermi energy lambda_f is the root of the
// electron-count constraint 2 sum_n g_n = N_e (Eq.
// FermiEnergyConstraintFormulation), g_n the Fermi-Dirac occupation of Ritz
// value theta_n at smearing k_B T.  It is found on the host by Brent's method
// (the paper's choice, Sec. 4) over N_s scalars; no device work is involved.
//
// The density rho = (2/h^3) sum_n g_n psi_n^2 is one streaming pass over the
// rotated block: every lane owns one 16-byte run of grid points (4 FP32 or 2
// FP64 values), walks the N_s columns in ascending order with eight column
// loads in flight, and accumulates in FP64, so the result does not depend on
// the launch shape.  The pass reads s N_d N_s bytes and writes 8 N_d; it is
// bound by HBM bandwidth.
#include <algorithm>
#include <cfloat>
#include <cmath>

#include "internal.hpp"

namespace sparc {
namespace {

// The constraint 2 sum g_n - N_e, evaluated without cancellation: with
// n_below levels at or below l, it equals
//   2 ((n_below - N_e/2) + sum_{theta > l} g_n - sum_{theta <= l} (1 - g_n)),
// and both kinds of tail term are exp(-|theta - l|/kT) / (1 + exp(...)), so
// they stay accurate (down to underflow) however far the level lies from l.
double count_residual(const double *theta, int ns, double ne, double kT, double l)
{
    long below = 0;
    double above_tail = 0.0, below_tail = 0.0;
    for (int n = 0; n < ns; ++n) {
        const double d = theta[n] - l;
        const double e = std::exp(-std::fabs(d) / kT);
        const double t = e / (1.0 + e);
        if (d > 0) {
            above_tail += t;
        } else {
            ++below;
            below_tail += t;
        }
    }
    return 2.0 * (((double)below - 0.5 * ne) + (above_tail - below_tail));
}

// Brent's root finder (inverse quadratic interpolation, secant and bisection
// steps, keeping a sign-changing bracket [b, c]; R. P. Brent, Algorithms for
// Minimization without Derivatives, 1973, ch. 4).  f(lo) < 0 < f(hi).
template <typename F>
double brent_root(F f, double lo, double hi, double flo, double fhi, double abs_tol)
{
    double a = lo, fa = flo, b = hi, fb = fhi;
    double c = a, fc = fa, step = b - a, prev_step = step;
    for (int it = 0; it < 300; ++it) {
        if ((fb > 0) == (fc > 0)) {  // keep the root between b and c
            c = a;
            fc = fa;
            step = prev_step = b - a;
        }
        if (std::fabs(fc) < std::fabs(fb)) {  // b is the best estimate so far
            a = b;
            b = c;
            c = a;
            fa = fb;
            fb = fc;
            fc = fa;
        }
        const double tol = 2.0 * DBL_EPSILON * std::fabs(b) + 0.5 * abs_tol;
        const double half = 0.5 * (c - b);
        if (std::fabs(half) <= tol || fb == 0.0) return b;
        if (std::fabs(prev_step) >= tol && std::fabs(fa) > std::fabs(fb)) {
            // interpolate: secant through (a, b), or an inverse quadratic
            // through a, b and c when all three differ
            double p, q;
            const double s = fb / fa;
            if (a == c) {
                p = 2.0 * half * s;
                q = 1.0 - s;
            } else {
                const double qa = fa / fc, r = fb / fc;
                p = s * (2.0 * half * qa * (qa - r) - (b - a) * (r - 1.0));
                q = (qa - 1.0) * (r - 1.0) * (s - 1.0);
            }
            if (p > 0)
                q = -q;
            else
                p = -p;
            // accept the interpolated point only if it falls well inside the
            // bracket and the steps keep shrinking; otherwise bisect
            if (2.0 * p < std::min(3.0 * half * q - std::fabs(tol * q), std::fabs(prev_step * q))) {
                prev_step = step;
                step = p / q;
            } else {
                step = prev_step = half;
            }
        } else {
            step = prev_step = half;
        }
        a = b;
        fa = fb;
        b += std::fabs(step) > tol ? step : (half > 0 ? tol : -tol);
        fb = f(b);
    }
    return b;
}

template <typename T>
struct DenVec;
template <>
struct DenVec<float> {
    typedef float V __attribute__((ext_vector_type(4)));
    static constexpr int N = 4;
};
template <>
struct DenVec<double> {
    typedef double V __attribute__((ext_vector_type(2)));
    static constexpr int N = 2;
};

constexpr int kDenUnroll = 8;  // column loads in flight per lane

// accumulates one column's values at a lane's N points, columns ascending
template <int N, typename V>
__device__ __forceinline__ void den_add(double (&acc)[N], const V &x, double g)
{
#pragma unroll
    for (int p = 0; p < N; ++p) {
        const double v = (double)x[p];
        acc[p] += g * v * v;
    }
}

// rho[i] = scale * sum_n occ[n] * psi_n[i]^2, columns in ascending order, one
// 16-byte load per lane and column.  Blocks whose columns all start on 16 bytes
// (SHIFT = false): lane t owns points [N t, N t + N).  Others (odd grids, padded
// leading dimensions): a 16-byte load off its alignment is split and reached
// 4.4 TB/s, so a lane loads the aligned unit its points start in and takes the
// rest from the next lane's; the 64th lane of a wave only lends its unit, a wave
// owns 63 N points.  The offset within the unit is the same for a whole column.
// NT: blocks the last-level cache cannot hold are read non-temporally.
// Measured (blocks not in cache): 127 x 119 x 131 x 256 FP32 546 us by scalar
// loads, 463 us by unaligned ones, 364 to 388 us now (5.6 TB/s); 99 x 101 x 103
// x 128 FP64 193 -> 173 us (by units shifted like the FP32 ones 184); aligned 160^3 x 600 FP32 1.82 -> 1.68 ms (5.9 TB/s).
template <typename T, bool NT, bool SHIFT>
__global__ void __launch_bounds__(512)
    density_kernel(const T *__restrict__ psi, long long ld, long long nd, int ns, const double *__restrict__ occ,
                   double scale, double *__restrict__ rho)
{
    constexpr int N = DenVec<T>::N;
    using V = typename DenVec<T>::V;
    typedef T VU __attribute__((ext_vector_type(N), aligned(sizeof(T))));
    const int lane = threadIdx.x & 63;
    const long long wave = (long long)blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6);
    const long long i0 = SHIFT ? (wave * 63 + lane) * N : (wave * 64 + lane) * N;
    double acc[N];
#pragma unroll
    for (int p = 0; p < N; ++p) acc[p] = 0.0;
    if (!SHIFT && i0 + N <= nd) {
        const T *col = psi + i0;
        int n = 0;
        for (; n + kDenUnroll <= ns; n += kDenUnroll) {
            V x[kDenUnroll];
#pragma unroll
            for (int j = 0; j < kDenUnroll; ++j) {
                const VU *c = (const VU *)(col + (long long)(n + j) * ld);
                x[j] = NT ? __builtin_nontemporal_load(c) : *c;
            }
#pragma unroll
            for (int j = 0; j < kDenUnroll; ++j) den_add<N>(acc, x[j], occ[n + j]);
        }
        for (; n < ns; ++n) {
            const V x = *(const VU *)(col + (long long)n * ld);
            den_add<N>(acc, x, occ[n]);
        }
    } else if (SHIFT) {
        if (wave * 63 * N >= nd) return;  // the whole wave
        const long long last = (long long)(ns - 1) * ld + nd;  // elements of the block
        const int ph = (int)(((uintptr_t)psi / sizeof(T)) % N);
        for (int n0 = 0; n0 < ns; n0 += kDenUnroll) {
            V x[kDenUnroll];
            int sh[kDenUnroll];
#pragma unroll
            for (int j = 0; j < kDenUnroll; ++j) {
                const int n = n0 + j < ns ? n0 + j : ns - 1;
                sh[j] = (int)((ph + (long long)n * ld) % N);
                const long long e = (long long)n * ld + i0 - sh[j];  // the aligned unit
                if (e >= 0 && e + N <= last) {
                    const V *c = (const V *)(psi + e);
                    x[j] = NT ? __builtin_nontemporal_load(c) : *c;
                } else {
#pragma unroll
                    for (int p = 0; p < N; ++p) x[j][p] = e + p >= 0 && e + p < last ? psi[e + p] : T(0);
                }
            }
#pragma unroll
            for (int j = 0; j < kDenUnroll; ++j) {
                if (n0 + j >= ns) break;
                T e[2 * N - 1];  // the lane's unit and the start of the next lane's
#pragma unroll
                for (int p = 0; p < N; ++p) e[p] = x[j][p];
#pragma unroll
                for (int p = 0; p + 1 < N; ++p) e[N + p] = __shfl_down(x[j][p], 1);
                V v = x[j];
#pragma unroll
                for (int d = 1; d < N; ++d)
                    if (sh[j] == d) {
#pragma unroll
                        for (int p = 0; p < N; ++p) v[p] = e[p + d];
                    }
                den_add<N>(acc, v, occ[n0 + j]);
            }
        }
        if (lane == 63) return;
    } else {
        for (int n = 0; n < ns; ++n) {
            V x;
#pragma unroll
            for (int p = 0; p < N; ++p) x[p] = i0 + p < nd ? psi[(long long)n * ld + i0 + p] : T(0);
            den_add<N>(acc, x, occ[n]);
        }
    }
    // whole units in 16-byte stores (rho starts on any double): for one column
    // the writes are two thirds of the traffic
    typedef double D2 __attribute__((ext_vector_type(2), aligned(sizeof(double))));
    if (i0 + N <= nd) {
#pragma unroll
        for (int p = 0; p < N; p += 2) *(D2 *)(rho + i0 + p) = D2{scale * acc[p], scale * acc[p + 1]};
    } else {
#pragma unroll
        for (int p = 0; p < N; ++p)
            if (i0 + p < nd) rho[i0 + p] = scale * acc[p];
    }
}

// FP64 columns off the 16-byte grid: a lane owns the points l and l + 64 of its
// wave's 128, so that its 8-byte loads are whole lines of the wave wherever a
// column starts.  U columns in flight; WHOLE: groups of U columns first (few
// waves need all their loads at once, 45 x 47 x 43 x 100 13.3 us, without 32;
// blocks from memory are faster without, 127 x 119 x 131 x 256 597 us, 697).
template <bool NT, bool WHOLE, int U>
__global__ void __launch_bounds__(512)
    density_split_kernel(const double *__restrict__ psi, long long ld, long long nd, int ns,
                         const double *__restrict__ occ, double scale, double *__restrict__ rho)
{
    const long long wave = (long long)blockIdx.x * (blockDim.x / 64) + (threadIdx.x >> 6);
    const long long i0 = wave * 128 + (threadIdx.x & 63), i1 = i0 + 64;
    if (i0 >= nd) return;
    const double *c0 = psi + i0, *c1 = psi + (i1 < nd ? i1 : i0);
    double acc[2] = {0.0, 0.0};
    typedef double V __attribute__((ext_vector_type(2)));
    int n0 = 0;
    if (WHOLE)
        for (; n0 + U <= ns; n0 += U) {
            V x[U];
#pragma unroll
            for (int j = 0; j < U; ++j) x[j] = V{c0[(long long)(n0 + j) * ld], c1[(long long)(n0 + j) * ld]};
#pragma unroll
            for (int j = 0; j < U; ++j) den_add<2>(acc, x[j], occ[n0 + j]);
        }
    for (; n0 < ns; n0 += U) {
        V x[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const long long o = (long long)min(n0 + j, ns - 1) * ld;
            x[j][0] = NT ? __builtin_nontemporal_load(c0 + o) : c0[o];
            x[j][1] = NT ? __builtin_nontemporal_load(c1 + o) : c1[o];
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            if (n0 + j >= ns) break;
            den_add<2>(acc, x[j], occ[n0 + j]);
        }
    }
    rho[i0] = scale * acc[0];
    if (i1 < nd) rho[i1] = scale * acc[1];
}

template <typename T>
int launch_density(const T *psi, long long ld, long long nd, int ns, const double *occ, double scale, double *rho,
                   hipStream_t s)
{
    constexpr int N = DenVec<T>::N;
    // Columns off the 16-byte grid: FP32 as aligned units shifted across the lanes,
    // FP64 point by point (density_split_kernel).
    const bool nt_loads = (double)nd * ns * sizeof(T) > kStreamBytes;
    const bool aligned = ld % N == 0 && (uintptr_t)psi % 16 == 0;
    const bool split = sizeof(T) == 8 && !aligned;
    const long long per = (aligned || split ? 64LL : 63LL) * N;  // points per wave
    const long long waves = (nd + per - 1) / per;
    // workgroups of 8 waves; small grids spread over more CUs by waves of their own
    const int nt = waves >= 4096 ? 512 : split ? 256 : 64;
    const long long blocks = (waves * 64 + nt - 1) / nt;
    if (blocks > 0x7fffffffLL) return fail(SPARC_E_SHAPE, "grid too large for one density launch");
    ProfScope prof(4, s);
#define SPARC_DEN(A, B)                                                                                            \
    hipLaunchKernelGGL((density_kernel<T, A, B>), dim3((unsigned)blocks), dim3(nt), 0, s, psi, ld, nd, ns, occ, scale, rho)
    if (aligned && nt_loads) {
        SPARC_DEN(true, false);
    } else if (aligned) {
        SPARC_DEN(false, false);
    } else if constexpr (sizeof(T) == 4) {
        if (nt_loads)
            SPARC_DEN(true, true);
        else
            SPARC_DEN(false, true);
    } else {
        // in the last-level cache a full chip needs few loads per lane: 95 x 97 x
        // 91 x 40 columns 42.6 us by two, 44.5 by eight; 45 x 47 x 43 x 100 19.7
        // and 13.3; from memory 127 x 119 x 131 x 20 57.9 and 51.6
#define SPARC_DEN_SPLIT(A, W, U)                                                                                  \
    hipLaunchKernelGGL((density_split_kernel<A, W, U>), dim3((unsigned)blocks), dim3(nt), 0, s, psi, ld, nd, ns, occ, \
                       scale, rho)
        if (nt_loads)
            SPARC_DEN_SPLIT(true, false, 8);
        else if (waves >= 4096)
            SPARC_DEN_SPLIT(false, false, 2);
        else
            SPARC_DEN_SPLIT(false, true, 8);
#undef SPARC_DEN_SPLIT
    }
#undef SPARC_DEN
    SPARC_HIP(hipGetLastError());
    return SPARC_OK;
}

}  // namespace
}  // namespace sparc

using namespace sparc;

extern "C" int sparc_fermi_level(const double *theta, int32_t ns, double ne, double kT, double *lambda_f, double *occ)
{
    if (!theta || !lambda_f || ns < 1) return fail(SPARC_E_ARG, "bad arguments");
    if (!(kT > 0.0) || !std::isfinite(kT)) return fail(SPARC_E_ARG, "k_B T must be positive");
    if (!(ne > 0.0 && ne < 2.0 * ns)) return fail(SPARC_E_ARG, "need 0 < N_e < 2 N_s");
    double tmin = theta[0], tmax = theta[0];
    for (int n = 0; n < ns; ++n) {
        if (!std::isfinite(theta[n])) return fail(SPARC_E_ARG, "non-finite eigenvalue");
        tmin = std::min(tmin, theta[n]);
        tmax = std::max(tmax, theta[n]);
    }
    auto f = [&](double l) { return count_residual(theta, ns, ne, kT, l); };
    // the residual rises monotonically from -N_e to 2 N_s - N_e: widen a
    // bracket around the spectrum until it changes sign
    double lo = tmin - 40.0 * kT, hi = tmax + 40.0 * kT;
    double flo = f(lo), fhi = f(hi);
    for (int k = 0; k < 64 && flo >= 0; ++k) flo = f(lo -= 40.0 * kT * (1 << std::min(k, 20)));
    for (int k = 0; k < 64 && fhi <= 0; ++k) fhi = f(hi += 40.0 * kT * (1 << std::min(k, 20)));
    if (flo >= 0 || fhi <= 0) return fail(SPARC_E_BOUNDS, "no sign change of the electron-count residual");
    const double lf = brent_root(f, lo, hi, flo, fhi, 1e-15 * kT);
    *lambda_f = lf;
    if (occ)
        for (int n = 0; n < ns; ++n) {
            const double x = (theta[n] - lf) / kT;
            occ[n] = x > 0 ? std::exp(-x) / (1.0 + std::exp(-x)) : 1.0 / (1.0 + std::exp(x));
        }
    return SPARC_OK;
}

extern "C" int sparc_density(int32_t dtype, const void *psi, int64_t ld, int64_t nd, int32_t ns, const double *occ,
                             double h, double *rho, void *stream)
{
    if (!psi || !occ || !rho || ns < 1 || (dtype != SPARC_F64 && dtype != SPARC_F32))
        return fail(SPARC_E_ARG, "bad arguments");
    if (nd < 1 || ld < nd || !(h > 0.0)) return fail(SPARC_E_SHAPE, "need nd >= 1, ld >= nd, h > 0");
    const size_t es = elem_size(dtype);
    const char *p0 = (const char *)psi, *p1 = p0 + ((size_t)(ns - 1) * ld + nd) * es;
    const char *r0 = (const char *)rho, *r1 = r0 + (size_t)nd * sizeof(double);
    if (p0 < r1 && r0 < p1) return fail(SPARC_E_ALIAS, "rho overlaps the orbital block");
    const double scale = 2.0 / (h * h * h);
    TraceRange trace("sparc_density");
    hipStream_t s = (hipStream_t)stream;
    return dtype == SPARC_F64 ? launch_density((const double *)psi, ld, nd, ns, occ, scale, rho, s)
                              : launch_density((const float *)psi, ld, nd, ns, occ, scale, rho, s);
}
