// FP64 spectral-bound Lanczos, Rayleigh-Ritz projection and subspace rotation.
//
// Lanczos (Sec. 4: extremal eigenvalues of H by a few Lanczos iterations)
// runs entirely on the device: H v through the fused step kernel, then
// deterministic two-pass reductions for the inner products (one partial per
// block, then one fixed-order sum, finished by whichever kernel needs the
// value), and partial re-orthogonalisation against the stored basis, decided
// on the device by the omega recurrence.  The scalars stay on the device
// between steps, so the k steps are enqueued without host round trips; the
// tridiagonal T_k is copied back once and its eigenvalues are found on the
// host by Sturm-sequence bisection.
//
// Rayleigh-Ritz (Sec. 3.4, Eq. SubspaceGeneralizedEigenproblem): H Y is
// formed in FP64 by the fused kernels (an FP32 block is widened as it is
// loaded), H_s = Y^T (H Y) and M_s = Y^T Y come from one FP64 matrix-core
// kernel, and the symmetric-definite problem is solved on the device: in one
// workgroup (Cholesky + Jacobi) for up to 64 columns, beyond by rocSOLVER's
// Cholesky and divide-and-conquer eigensolver with the reduction to standard
// form and the back-transformation as rocBLAS triangular solves.
#include <rocblas/rocblas.h>
#include <rocsolver/rocsolver.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <map>
#include <type_traits>
#include <vector>

#include "internal.hpp"

namespace sparc {

thread_local bool g_rr_rank_deficient = false;  // set by the last Rayleigh-Ritz call of this thread

constexpr int kDotGroup = 8;      // vectors per pass over a block's segment
constexpr int kUnroll = 4;        // points per thread with loads in flight together

__device__ inline double wave_sum(double v)
{
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// sum over the 4 waves of a 256-thread block, the same value in every thread
__device__ inline double block_sum(double v, double *red)
{
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    const double t = (red[0] + red[1]) + (red[2] + red[3]);
    __syncthreads();
    return t;
}

// sum of entry i of the kRedBlocks block partials (stride per block) in one
// fixed order, so that every block that needs the value finishes it
// bitwise identically
__device__ inline double sum_partials(const double *partial, int stride, int i, double *red)
{
    double v = 0.0;
#pragma unroll
    for (int u = 0; u < kRedBlocks / 256; ++u) v += partial[(long long)(threadIdx.x + 256 * u) * stride + i];
    return block_sum(v, red);
}

// the contiguous segment of n points owned by block b of a reduction pass
__device__ inline void block_segment(long long n, long long &beg, long long &end)
{
    const long long seg = red_segment(n);
    beg = blockIdx.x * seg;
    end = (beg + seg < n) ? beg + seg : n;
}

// per-block partials of |w|^2
__global__ void __launch_bounds__(256) norm2_kernel(const double *__restrict__ w, long long n,
                                                    double *__restrict__ partial)
{
    __shared__ double red[4];
    long long beg, end;
    block_segment(n, beg, end);
    double s = 0.0;
    for (long long x0 = beg + threadIdx.x; x0 < end; x0 += 256 * kUnroll)
#pragma unroll
        for (int r = 0; r < kUnroll; ++r) {
            const long long x = x0 + 256 * r;
            const double v = x < end ? w[x] : 0.0;
            s += v * v;
        }
    s = block_sum(s, red);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// The Lanczos vectors are kept as they come out of the recurrence, u_j = nu_j
// v_j with nu_j = |u_j| = beta_{j-1} (nu_0 = 1): nothing is scaled in a pass of
// its own.
//
// alpha_j = v_j^T H v_j from its two parts: the step kernel's workgroup
// partials of u^T (H_loc u), and the projections g_p = chi_p^T u (the gather's
// split partials, nproj of them per split), since u^T V_nl u = sum_p hg_p
// g_p^2.  table (LDS, may be null) receives hg_p g_p.  nu_j is finished first
// when the step before re-orthogonalised u_j (its |u_j|^2 partials).  One fixed
// order in every block.
struct LanczosAlpha {
    const double *dot;
    int ndot;
    const double *gpart, *hg;
    int nproj;
    const int *redo;      // u_j was re-orthogonalised (null: never)
    const double *npart;  // then: partials of |u_j|^2
};

__device__ inline double lanczos_alpha(const LanczosAlpha &q, double *nu_j, double *table, double *red, double &nu)
{
    double v = 0.0;
    for (int b = threadIdx.x; b < q.ndot; b += 256) v += q.dot[b];
    for (int p = threadIdx.x; p < q.nproj; p += 256) {
        double g = 0.0;
#pragma unroll
        for (int s = 0; s < kGatherSplit; ++s) g += q.gpart[(long long)s * q.nproj + p];
        const double t = q.hg[p] * g;
        if (table) table[p] = t;
        v += t * g;
    }
    v = block_sum(v, red);
    nu = *nu_j;
    if (q.redo && *q.redo) {
        nu = sqrt(sum_partials(q.npart, 1, 0, red));
        if (blockIdx.x == 0 && threadIdx.x == 0) *nu_j = nu;
    }
    return v / (nu * nu);
}

__global__ void __launch_bounds__(256) alpha_finish(const LanczosAlpha q, double *nu_j, double *alpha)
{
    __shared__ double red[4];
    double nu;
    const double a = lanczos_alpha(q, nu_j, nullptr, red, nu);
    if (threadIdx.x == 0) *alpha = a;
}

// nonlocal nodes of a reduction segment (see scatter_item for the tables):
// block b's segment covers entries seg[b] .. seg[b+1] of pts
struct LanczosScatter {
    const int *seg;
    const int *pts, *ent_off;
    const int4 *ent;
    const int *ent_proj;  // first projector of each entry's atom
    const double *chi;
};

constexpr int kLanczosProj = 2048;  // projectors whose table the fused scatter keeps in LDS (16 KiB)

// Three-term step: on entry w = H_loc u_j.  The projector scatter of the
// block's own nodes comes first (FUSED: w += V_nl u_j, the sums of
// scatter_item; otherwise the scatter was a launch of its own), then
//   w <- w / nu_j - (alpha_j / nu_j) u_j - (beta_{j-1} / nu_{j-1}) u_{j-1}
// and partial[b] = sum over block b's nodes of the new w^2.
// What bounds it: the chain of dependent launches.  A step takes four (H u with
// the projections, this one, the orthogonality estimates, the conditional
// re-orthogonalisation) where it took seven (scatter, sums and scaling apart).
template <bool FUSED>
__global__ void __launch_bounds__(256)
    lanczos_3term(double *w, const double *__restrict__ uj, const double *__restrict__ ujm, const LanczosAlpha q,
                  const LanczosScatter sc, double *nu_j, double *alpha, long long n, double *__restrict__ partial)
{
    __shared__ double red[4];
    __shared__ double table[FUSED ? kLanczosProj : 1];
    // what the sums do not decide is requested before them: the thread's first
    // nodes of u_j and u_{j-1}, and its first nonlocal node
    long long beg, end;
    block_segment(n, beg, end);
    const double *um = ujm ? ujm : uj;
    double v1[kUnroll], v2[kUnroll];
#pragma unroll
    for (int r = 0; r < kUnroll; ++r) {
        const long long x = beg + threadIdx.x + 256 * r;
        v1[r] = x < end ? uj[x] : 0.0;
        v2[r] = x < end ? um[x] : 0.0;
    }
    int pi = 0, pe = 0, node = 0, e0 = 0, e1 = 0, pj = 0;
    int4 en = make_int4(0, 0, 0, 0);
    if (FUSED) {
        pi = sc.seg[blockIdx.x] + threadIdx.x;
        pe = sc.seg[blockIdx.x + 1];
        if (pi < pe) {
            node = sc.pts[pi];
            e0 = sc.ent_off[pi];
            e1 = sc.ent_off[pi + 1];
            en = sc.ent[e0];
            pj = sc.ent_proj[e0];
        }
    }
    double nu;
    const double a = lanczos_alpha(q, nu_j, FUSED ? table : nullptr, red, nu);
    if (blockIdx.x == 0 && threadIdx.x == 0) *alpha = a;
    if (FUSED) {  // table complete: block_sum ends in a barrier
        while (pi < pe) {
            const double cur = w[node];
            double acc = 0.0;
            for (int e = e0; e < e1; ++e) {
                if (e > e0) {
                    en = sc.ent[e];
                    pj = sc.ent_proj[e];
                }
                const double *S = table + pj;
                for (int p = 0; p < en.w; ++p) acc += sc.chi[en.x + (long long)p * en.y] * S[p];
            }
            w[node] = cur + acc;
            pi += 256;
            if (pi < pe) {
                node = sc.pts[pi];
                e0 = sc.ent_off[pi];
                e1 = sc.ent_off[pi + 1];
                en = sc.ent[e0];
                pj = sc.ent_proj[e0];
            }
        }
        __syncthreads();
    }
    const double c0 = 1.0 / nu, c1 = a / nu, c2 = ujm ? nu / nu_j[-1] : 0.0;
    double nrm = 0.0;
    for (long long x0 = beg + threadIdx.x; x0 < end; x0 += 256 * kUnroll) {
        double wv[kUnroll];
#pragma unroll
        for (int r = 0; r < kUnroll; ++r) {
            const long long x = x0 + 256 * r;
            const bool ok = x < end;
            wv[r] = ok ? w[x] : 0.0;
            if (x0 >= beg + 256 * kUnroll) {
                v1[r] = ok ? uj[x] : 0.0;
                v2[r] = ok ? um[x] : 0.0;
            }
        }
#pragma unroll
        for (int r = 0; r < kUnroll; ++r) {
            const long long x = x0 + 256 * r;
            if (x < end) {
                const double v = c0 * wv[r] - (c1 * v1[r] + c2 * v2[r]);
                w[x] = v;
                nrm += v * v;
            }
        }
    }
    const double t = block_sum(nrm, red);
    if (threadIdx.x == 0) partial[blockIdx.x] = t;
}

constexpr int kDotBlocks = 256;  // workgroups of the inner products: few partials for every workgroup to finish

// Partial reorthogonalisation (Simon's omega recurrence).  Row j of the
// estimates holds v_j^T v_i, i < j; after the three-term step of step j
// (coefficients alpha_j and beta_j), for i < j
//   beta_j w'_i = beta_i w_{i+1} + (alpha_i - alpha_j) w_i + beta_{i-1} w_{i-1}
//                 - beta_{j-1} w''_i  (+ eps1 (beta_i + beta_j) for rounding),
// w = row j, w'' = row j-1, and w'_j = eps1 ||T|| / beta_j.  The new vector
// is orthogonalised against the whole basis when an estimate passes sqrt(eps)
// and, after that, once more on the next step; its row then restarts at eps1.
//
// Every workgroup of this kernel finishes beta_j = sqrt(sum of the block
// partials of |w|^2) (the same fixed order as finish_sums) and evaluates the
// recurrence and the decision itself, bitwise identically; workgroup 0 stores
// beta_j, row j+1, ||T|| (anorm[j+1]), full[j] (orthogonalise now) and
// owed[j+1] (orthogonalise the next vector too).  Per-step slots keep the
// values read (owed[j], anorm[j]) apart from those written.  When the
// vector is to be orthogonalised, the workgroups go on to the inner products
// u_i^T w, i = 0 .. j (the first kDotBlocks workgroups, partial[i][block]);
// otherwise they exit.
__global__ void __launch_bounds__(256) omega_dots_kernel(const double *alpha, double *beta, int j, double eps1,
                                                         const double *Wp, const double *Wc, double *Wn,
                                                         int *owed, int *full, double *anorm,
                                                         const double *npart, const double *__restrict__ V,
                                                         long long ldv, const double *__restrict__ w, long long n,
                                                         double *__restrict__ partial)
{
    __shared__ double red[4];
    __shared__ int sfull;
    const double bj = sqrt(sum_partials(npart, 1, 0, red));
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x;
        const double aj = alpha[j], bjm = j > 0 ? beta[j - 1] : 0.0;
        const double an = fmax(anorm[j], fabs(aj) + bj + bjm);
        double mx = 0.0;
        for (int i = lane; i < j; i += 64) {
            double t = beta[i] * Wc[i + 1] + (alpha[i] - aj) * Wc[i] - bjm * Wp[i];
            if (i > 0) t += beta[i - 1] * Wc[i - 1];
            t += copysign(eps1 * (beta[i] + bj), t);
            mx = fmax(mx, fabs(t / bj));
        }
        for (int off = 32; off > 0; off >>= 1) mx = fmax(mx, __shfl_xor(mx, off));
        const double dj = eps1 * an / bj;
        const bool owe = owed[j] != 0;
        const bool f = owe || fmax(mx, dj) > 1.4901161193847656e-08;  // sqrt(eps)
        if (blockIdx.x == 0) {
            // second pass for the row values (cheap, avoids holding them across the reduction)
            for (int i = lane; i < j; i += 64) {
                double t = beta[i] * Wc[i + 1] + (alpha[i] - aj) * Wc[i] - bjm * Wp[i];
                if (i > 0) t += beta[i - 1] * Wc[i - 1];
                t += copysign(eps1 * (beta[i] + bj), t);
                Wn[i] = f ? eps1 : t / bj;
            }
            if (lane == 0) {
                beta[j] = bj;
                Wn[j] = f ? eps1 : dj;
                Wn[j + 1] = 1.0;
                anorm[j + 1] = an;
                full[j] = f ? 1 : 0;
                owed[j + 1] = (f && !owe) ? 1 : 0;
            }
        }
        if (lane == 0) sfull = f ? 1 : 0;
    }
    __syncthreads();
    if (!sfull || blockIdx.x >= kDotBlocks) return;
    const long long seg = ((n + kDotBlocks - 1) / kDotBlocks + 63) / 64 * 64;
    const long long beg = blockIdx.x * seg, end = beg + seg < n ? beg + seg : n;
    const int nv = j + 1;
    for (int i0 = 0; i0 < nv; i0 += kDotGroup) {
        double acc[kDotGroup];
#pragma unroll
        for (int u = 0; u < kDotGroup; ++u) acc[u] = 0.0;
        for (long long x0 = beg + threadIdx.x; x0 < end; x0 += 256 * kUnroll) {
            double wx[kUnroll];
#pragma unroll
            for (int r = 0; r < kUnroll; ++r) {
                const long long x = x0 + 256 * r;
                wx[r] = x < end ? w[x] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < kDotGroup; ++u) {
                const int i = i0 + u;
                if (i >= nv) break;
                double vx[kUnroll];
#pragma unroll
                for (int r = 0; r < kUnroll; ++r) {
                    const long long x = x0 + 256 * r;
                    vx[r] = x < end ? V[(long long)i * ldv + x] : 0.0;
                }
#pragma unroll
                for (int r = 0; r < kUnroll; ++r) acc[u] += vx[r] * wx[r];
            }
        }
#pragma unroll
        for (int u = 0; u < kDotGroup; ++u) {
            const double t = block_sum(acc[u], red);
            if (threadIdx.x == 0 && i0 + u < nv) partial[(long long)(i0 + u) * kDotBlocks + blockIdx.x] = t;
        }
    }
}

constexpr int kOrthPanel = 1024;  // coefficients in LDS at a time: the step count has no limit

// where the decision (run) asks for it: c_i = u_i^T w / nu_i^2 from the
// partials (every workgroup in the same fixed order, one wave per c_i), w -=
// sum_i c_i u_i by panels of kOrthPanel vectors, and partial[b] = sum over
// block b's nodes of the new w^2
__global__ void __launch_bounds__(256) orth_apply_norm(double *w, const double *__restrict__ V, long long ldv, int nv,
                                                       const double *__restrict__ dots, const double *__restrict__ nu,
                                                       long long n, double *__restrict__ partial, const int *run)
{
    __shared__ double coeff[kOrthPanel];
    if (!*run) return;
    __shared__ double red[4];
    long long beg, end;
    block_segment(n, beg, end);
    double nrm = 0.0;
    for (int p0 = 0; p0 < nv; p0 += kOrthPanel) {
        const int np = min(kOrthPanel, nv - p0);
        const bool last = p0 + np == nv;
        if (p0 > 0) __syncthreads();
        for (int i = threadIdx.x >> 6; i < np; i += 4) {
            double v = 0.0;
#pragma unroll
            for (int u = 0; u < kDotBlocks / 64; ++u)
                v += dots[(long long)(p0 + i) * kDotBlocks + 64 * u + (threadIdx.x & 63)];
            v = wave_sum(v);
            if ((threadIdx.x & 63) == 0) coeff[i] = v / (nu[p0 + i] * nu[p0 + i]);
        }
        __syncthreads();
        for (long long x0 = beg + threadIdx.x; x0 < end; x0 += 256 * kUnroll) {
            double s[kUnroll];
#pragma unroll
            for (int r = 0; r < kUnroll; ++r) s[r] = 0.0;
            for (int i = 0; i < np; ++i) {
                const double c = coeff[i];
#pragma unroll
                for (int r = 0; r < kUnroll; ++r) {
                    const long long x = x0 + 256 * r;
                    s[r] += c * (x < end ? V[(long long)(p0 + i) * ldv + x] : 0.0);
                }
            }
#pragma unroll
            for (int r = 0; r < kUnroll; ++r) {
                const long long x = x0 + 256 * r;
                if (x < end) {
                    const double v = w[x] - s[r];
                    w[x] = v;
                    if (last) nrm += v * v;
                }
            }
        }
    }
    const double t = block_sum(nrm, red);
    if (threadIdx.x == 0) partial[blockIdx.x] = t;
}

// rows j = 0 (1 at i = 0) and j = -1 (zero); owed[0] = 0, anorm[0] = 0,
// nu[0] = 1
__global__ void omega_init(double *rows, int len, int *owed, double *anorm, double *nu)
{
    for (int i = threadIdx.x; i < 3 * len; i += blockDim.x) rows[i] = (i == 0) ? 1.0 : 0.0;
    if (threadIdx.x == 0) {
        owed[0] = 0;
        *anorm = 0.0;
        nu[0] = 1.0;
    }
}

// dst = src / |src|, |src|^2 from its block partials
__global__ void __launch_bounds__(256) scale_by_norm(double *dst, const double *__restrict__ src,
                                                     const double *partial, long long n)
{
    __shared__ double red[4];
    const double inv = 1.0 / sqrt(sum_partials(partial, 1, 0, red));
    long long beg, end;
    block_segment(n, beg, end);
    for (long long x = beg + threadIdx.x; x < end; x += 256) dst[x] = src[x] * inv;
}

__global__ void f64_to_f32_dense(const double *src, float *dst, long long n)
{
    for (long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x; t < n; t += (long long)gridDim.x * blockDim.x)
        dst[t] = (float)src[t];
}

// ---------------------------------------------------------------- Rayleigh-Ritz projection
//
// M_s = Y^T Y and H_s = Y^T (HY) in FP64 on the matrix cores
// (v_mfma_f64_16x16x4f64).  The contraction runs over the N_d grid points,
// which are split into chunks; a workgroup owns one 64 x 64 tile pair of
// (M_s, H_s) on or above the diagonal for one chunk, stages 32-point slices of
// the three column panels in LDS (16 bytes per lane along the contiguous grid
// axis) and writes its part of the upper triangles, packed; a second kernel
// sums them in chunk order and writes both triangles.  The four waves share the
// 16 x 16 blocks of the tile that are on or above the diagonal and within ns,
// of both matrices (741 of the 880 in 55 whole tiles at ns = 600).  Workgroup
// indices are remapped so that all tile pairs of one chunk run on the same XCD.
//
// What bounds it: the matrix cores, busy 79 % of the time at 160^3 x 600 (FP32
// block): 53.3 ms, 62.7 with whole tiles and 4-byte loads; 45 with the loads
// taken out.  The panels come from the last-level cache (193 GB, the XCD's L2
// holds too few slices for the tile pairs of a chunk to meet in it), with a
// latency the next slice's loads cover.  Tiles of 128 halve those bytes but
// leave two waves per SIMD, one workgroup per CU: 62.8 ms.

constexpr int kRrTile = 64;
constexpr int kRrK = 32;  // points per staged slice; chunks of the contraction are multiples of it

// Staged slice: FP32 panels stay FP32 in LDS (widened when read as MFMA
// operands).  The row strides (36 floats, 34 doubles) keep the 16-byte writes
// aligned and put the 16 rows of one operand read in distinct banks.
template <typename TY>
struct RrPanels {
    static constexpr int SA = sizeof(TY) == 4 ? kRrK + 4 : kRrK + 2;
    alignas(16) TY A[kRrTile][SA];            // Y columns of the row tile, [col][k]
    alignas(16) TY B[kRrTile][SA];            // Y columns of the column tile
    alignas(16) double H[kRrTile][kRrK + 2];  // HY columns of the column tile
};

__device__ inline void mfma_f64(double a, double b, double (&acc)[4])
{
    typedef double v4d __attribute__((ext_vector_type(4)));
    v4d c = {acc[0], acc[1], acc[2], acc[3]};
    c = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    acc[0] = c[0];
    acc[1] = c[1];
    acc[2] = c[2];
    acc[3] = c[3];
}

// acc += the 16 x 16 blocks of one wave of a diagonal tile over a staged slice:
// the five blocks on and above the diagonal of block rows W and 3 - W of Y^T Y
// or, HY, of Y^T (H Y)
template <typename TY, int W, bool HY>
__device__ __forceinline__ void rr_diag(const RrPanels<TY> &S, int li, int lk, double (&acc)[8][4])
{
#pragma unroll
    for (int ks = 0; ks < kRrK; ks += 4) {
        const double a0 = (double)S.A[16 * W + li][ks + lk];
        const double a1 = (double)S.A[16 * (3 - W) + li][ks + lk];
#pragma unroll
        for (int v = W; v < 4; ++v) {
            const double b = HY ? S.H[16 * v + li][ks + lk] : (double)S.A[16 * v + li][ks + lk];
            mfma_f64(a0, b, acc[v - W]);
            if (v >= 3 - W) mfma_f64(a1, b, acc[1 + v]);
        }
    }
}

template <typename T, int N>
struct RrVec {
    typedef T type __attribute__((ext_vector_type(N)));
};

// N points from p[k] on; TAIL: zeros past point kl
template <int N, bool TAIL, typename T>
__device__ __forceinline__ typename RrVec<T, N>::type rr_load(const T *p, int k, int kl)
{
    typedef T V __attribute__((ext_vector_type(N), aligned(sizeof(T))));
    if (!TAIL) return *(const V *)(p + k);
    typename RrVec<T, N>::type v;
#pragma unroll
    for (int e = 0; e < N; ++e) {
        const T t = p[min(k + e, kl)];
        v[e] = k + e <= kl ? t : T(0);
    }
    return v;
}

// One tile pair over the points [k0, k1).  The 16 x 16 blocks a wave forms:
//  NC = 4, a whole tile pair: 2 x 2 blocks of both matrices,
//  NC = 1..3, one cut by the matrix's edge: a block row and its NC columns,
//  NC = 0, a diagonal one: see rr_diag.
template <typename TY, int NC>
__device__ __forceinline__ void rr_pair(const TY *__restrict__ Y, long long ldy, const double *__restrict__ HY,
                                        long long ldh, int ns, int ti, int tj, long long k0, long long k1,
                                        RrPanels<TY> &S, double *__restrict__ pm)
{
    constexpr int T = kRrTile, KS = kRrK;
    constexpr bool DIAG = NC == 0;
    // 16 bytes per lane: VY points of a Y column (TY_ lanes a column), 2 of an HY column
    constexpr int VY = 16 / sizeof(TY), LY = KS / VY, CY = 256 / LY, PY = T / CY;
    constexpr int LH = KS / 2, CH = 256 / LH, PH = T / CH;
    typedef typename RrVec<TY, VY>::type VecY;
    typedef typename RrVec<double, 2>::type VecH;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wi = (wave >> 1) * 32, wj = (wave & 1) * 32;
    const int w = wave >> 1, hy = wave & 1;
    const int li = lane & 15, lk = lane >> 4;
    double acc[8][4] = {};
    VecY ra[PY], rb[PY];  // raw values of the next slice (keeps the loads in flight)
    VecH rh[PH];

    // On a diagonal tile pair both Y panels are the same columns: read and
    // stage them once.  Columns past ns repeat the last one (the blocks' rows
    // and columns past ns are not stored), points past k1 are staged as zeros.
    const int cy = tid / LY, ky = tid % LY * VY, ch = tid / LH, kh = tid % LH * 2;
    auto fetch_slice = [&](long long kb, auto tail) {
        constexpr bool TAIL = decltype(tail)::value;
        const int kl = (int)(k1 - 1 - kb);
        // (made again for each slice: the twelve column addresses would not fit
        // beside the sums)
        int y = cy, h = ch;
        asm volatile("" : "+v"(y), "+v"(h));
#pragma unroll
        for (int pass = 0; pass < PY; ++pass) {
            const int ca = ti * T + pass * CY + y, cb = min(tj * T + pass * CY + y, ns - 1);
            if (!DIAG) ra[pass] = rr_load<VY, TAIL>(Y + kb + ca * ldy, ky, kl);
            rb[pass] = rr_load<VY, TAIL>(Y + kb + cb * ldy, ky, kl);
        }
#pragma unroll
        for (int pass = 0; pass < PH; ++pass)
            rh[pass] = rr_load<2, TAIL>(HY + kb + min(tj * T + pass * CH + h, ns - 1) * ldh, kh, kl);
    };
    auto fetch = [&](long long kb) {
        if (kb + KS <= k1)
            fetch_slice(kb, std::false_type());
        else
            fetch_slice(kb, std::true_type());
    };
    fetch(k0);
    for (long long kb = k0; kb < k1; kb += KS) {
        __syncthreads();
#pragma unroll
        for (int pass = 0; pass < PY; ++pass) {
            const int c = pass * CY + cy;
            *(VecY *)&S.A[c][ky] = DIAG ? rb[pass] : ra[pass];
            if (!DIAG) *(VecY *)&S.B[c][ky] = rb[pass];
        }
#pragma unroll
        for (int pass = 0; pass < PH; ++pass) *(VecH *)&S.H[pass * CH + ch][kh] = rh[pass];
        __syncthreads();
        if (kb + KS < k1) fetch(kb + KS);
        if constexpr (DIAG) {
            switch (wave) {
                case 0: rr_diag<TY, 0, false>(S, li, lk, acc); break;
                case 1: rr_diag<TY, 0, true>(S, li, lk, acc); break;
                case 2: rr_diag<TY, 1, false>(S, li, lk, acc); break;
                default: rr_diag<TY, 1, true>(S, li, lk, acc); break;
            }
        } else {
            constexpr int NR = NC == 4 ? 2 : 1, NV = NC == 4 ? 2 : NC;
            const int r0 = NC == 4 ? wi : 16 * wave, c0 = NC == 4 ? wj : 0;
#pragma unroll
            for (int ks = 0; ks < KS; ks += 4) {
                double a[NR], b[NV], h[NV];
#pragma unroll
                for (int u = 0; u < NR; ++u) a[u] = (double)S.A[r0 + 16 * u + li][ks + lk];
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    b[v] = (double)S.B[c0 + 16 * v + li][ks + lk];
                    h[v] = S.H[c0 + 16 * v + li][ks + lk];
                }
#pragma unroll
                for (int u = 0; u < NR; ++u)
#pragma unroll
                    for (int v = 0; v < NV; ++v) {
                        mfma_f64(a[u], b[v], acc[2 * (NV * u + v)]);
                        mfma_f64(a[u], h[v], acc[2 * (NV * u + v) + 1]);
                    }
            }
        }
    }
    // pm: the two upper triangles, packed by columns
    const long long tri = (long long)ns * (ns + 1) / 2;
    auto put = [&](const double (&v)[4], int r0, int c0, bool h) {
        const long long col = tj * T + c0 + (lane & 15);
        double *p = pm + (h ? tri : 0) + col * (col + 1) / 2;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = ti * T + r0 + (lane >> 4) + 4 * r;
            if (row <= col && col < ns) p[row] = v[r];
        }
    };
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        if (NC == 4) put(acc[q], wi + 16 * (q / 4), wj + 16 * (q / 2 % 2), q & 1);
        if (!DIAG && NC < 4 && q < 2 * NC) put(acc[q], 16 * wave, 16 * (q / 2), q & 1);
        if (DIAG && q < 5) {
            const bool first = q < 4 - w;
            put(acc[q], 16 * (first ? w : 3 - w), 16 * (first ? q + w : q - 1), hy);
        }
    }
}

template <typename TY>
__global__ void __launch_bounds__(256, 3)
    rr_project_kernel(const TY *__restrict__ Y, long long ldy, const double *__restrict__ HY, long long ldh,
                      long long nd, int ns, long long kchunk, double *__restrict__ partial)
{
    __shared__ RrPanels<TY> S;
    // (chunk, tile pair) from the XCD-contiguous workgroup order; tile pair
    // (ti <= tj) numbered in row order: both matrices are symmetric, so only
    // the upper tiles are formed
    const int nt = (ns + kRrTile - 1) / kRrTile;
    const int npairs = nt * (nt + 1) / 2;
    const int nb = (int)gridDim.x, wg = (int)blockIdx.x, xcd = wg & 7;
    const int t = xcd * (nb >> 3) + min(xcd, nb & 7) + (wg >> 3);
    const int chunk = t / npairs;
    int ti = 0, rem = t % npairs;
    while (rem >= nt - ti) {
        rem -= nt - ti;
        ++ti;
    }
    const int tj = ti + rem;
    const long long k0 = chunk * kchunk;
    const long long k1 = (k0 + kchunk < nd) ? k0 + kchunk : nd;
    double *pm = partial + (long long)chunk * ns * (ns + 1);
    switch (ti == tj ? 0 : min(4, (ns - tj * kRrTile + 15) / 16)) {  // block columns within ns
        case 0: rr_pair<TY, 0>(Y, ldy, HY, ldh, ns, ti, tj, k0, k1, S, pm); break;
        case 1: rr_pair<TY, 1>(Y, ldy, HY, ldh, ns, ti, tj, k0, k1, S, pm); break;
        case 2: rr_pair<TY, 2>(Y, ldy, HY, ldh, ns, ti, tj, k0, k1, S, pm); break;
        case 3: rr_pair<TY, 3>(Y, ldy, HY, ldh, ns, ti, tj, k0, k1, S, pm); break;
        default: rr_pair<TY, 4>(Y, ldy, HY, ldh, ns, ti, tj, k0, k1, S, pm); break;
    }
}

// Ms, Hs (column-major ns x ns) = sum over chunks of the partial tiles for the
// entries on and above the diagonal, each written to both triangles.  G lanes
// share an entry (chunks dealt round-robin, their sums added in lane order): a
// small matrix has few entries and many chunks, and one lane per entry walked
// them in 17 us for 8 columns of 24^3; 16 consecutive entries per group keep
// the loads whole lines.
template <int G>
__global__ void __launch_bounds__(256) rr_reduce_kernel(const double *partial, int nchunks, int ns, double *Ms,
                                                        double *Hs)
{
    constexpr int E = 256 / G;  // entries per workgroup
    __shared__ double sum[G][E];
    const long long tri = (long long)ns * (ns + 1) / 2;
    const long long e = blockIdx.x * (long long)E + threadIdx.x % E;
    const int g = threadIdx.x / E;
    const bool in = e < 2 * tri;
    const long long which = e >= tri ? 1 : 0, off = e - which * tri;
    double s = 0.0;
    if (in) {
#pragma unroll 16
        for (int c = g; c < nchunks; c += G) s += partial[((long long)c * 2 + which) * tri + off];
    }
    if (G > 1) {
        sum[g][threadIdx.x % E] = s;
        __syncthreads();
        if (g > 0) return;
        s = 0.0;
#pragma unroll
        for (int k = 0; k < G; ++k) s += sum[k][threadIdx.x % E];
    }
    if (!in) return;
    // off = col (col + 1) / 2 + row, row <= col
    int col = (int)((sqrt(8.0 * (double)off + 1.0) - 1.0) * 0.5);
    while ((long long)(col + 1) * (col + 2) / 2 <= off) ++col;
    while ((long long)col * (col + 1) / 2 > off) --col;
    const int row = (int)(off - (long long)col * (col + 1) / 2);
    double *A = which == 0 ? Ms : Hs;
    A[(long long)col * ns + row] = s;
    A[(long long)row * ns + col] = s;
}

static dim3 stream_grid(long long n)
{
    long long b = (n + 255) / 256;
    return dim3((unsigned)std::min<long long>(b, 4096));
}

// ---------------------------------------------------------------- rotation

// out(x, c) = sum_j Y(x, j) Q(j, c) for a block of RotTile::cols output
// columns.  One thread per grid point x: the row of Y is read in chunks of
// RotTile::k values (each load coalesced along x); Q comes as a zero-padded
// copy in the block's dtype, column-major with a leading dimension that is a
// multiple of the chunk, so Q(k0.., c) is contiguous and wave-uniform (scalar
// loads); each thread keeps the sums of its point in registers and every
// output column is written coalesced along x.  HBM-bound: Y is read once and
// out written once per column block.
template <typename T>
struct RotTile;
template <>
struct RotTile<float> {
    static constexpr int cols = 64, k = 16;
};
template <>
struct RotTile<double> {
    static constexpr int cols = 32, k = 16;
};

inline int rot_ldq(int ns) { return (ns + 15) / 16 * 16; }
template <typename T>
inline int rot_ncols(int ns)
{
    return (ns + RotTile<T>::cols - 1) / RotTile<T>::cols * RotTile<T>::cols;
}

// Qp(j, c) = Q(j, c) for j, c < ns, zero elsewhere (ldq x ncp, column-major)
template <typename T>
__global__ void pad_rotation(const double *__restrict__ Q, int ns, T *__restrict__ Qp, int ldq, int ncp)
{
    const long long total = (long long)ldq * ncp;
    for (long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x; e < total;
         e += (long long)gridDim.x * blockDim.x) {
        const int j = (int)(e % ldq), c = (int)(e / ldq);
        Qp[e] = (j < ns && c < ns) ? (T)Q[(long long)c * ns + j] : T(0);
    }
}

template <typename T>
__global__ void __launch_bounds__(256) rotate_kernel(const T *__restrict__ Y, long long ldy, const T *__restrict__ Qp,
                                                     int ldq, T *__restrict__ out, long long ldo, long long nd, int ns)
{
    constexpr int NC = RotTile<T>::cols, KC = RotTile<T>::k;
    const long long x = blockIdx.x * 256LL + threadIdx.x;
    const int c0 = blockIdx.y * NC;
    const long long xs = x < nd ? x : nd - 1;  // loads stay in bounds; the store is masked
    T acc[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[c] = T(0);
    for (int k0 = 0; k0 < ns; k0 += KC) {
        T y[KC];
#pragma unroll
        for (int j = 0; j < KC; ++j) y[j] = (k0 + j < ns) ? Y[(long long)(k0 + j) * ldy + xs] : T(0);
        const T *q = Qp + (long long)c0 * ldq + k0;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            T t = acc[c];
#pragma unroll
            for (int j = 0; j < KC; ++j) t += y[j] * q[(long long)c * ldq + j];
            acc[c] = t;
        }
    }
    if (x < nd) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
            if (c0 + c < ns) out[(long long)(c0 + c) * ldo + x] = acc[c];
    }
}

// The same sums for up to NC <= 16 columns straight from the FP64 rotation
// (rounded to T as it is read, wave-uniform): no padded copy and no products
// with padding.  24^3 x 8 FP64: 6 us instead of 13 + 3 us.
constexpr int kRotSmall = 16;
template <typename T, int NC>
__global__ void __launch_bounds__(256) rotate_small_kernel(const T *__restrict__ Y, long long ldy,
                                                           const double *__restrict__ Q, T *__restrict__ out,
                                                           long long ldo, long long nd, int ns)
{
    const long long x = blockIdx.x * 256LL + threadIdx.x;
    if (x >= nd) return;
    T y[NC];
#pragma unroll
    for (int j = 0; j < NC; ++j) y[j] = j < ns ? Y[(long long)j * ldy + x] : T(0);
#pragma unroll 2
    for (int c = 0; c < ns; ++c) {
        T t = T(0);
#pragma unroll
        for (int j = 0; j < NC; ++j) t += y[j] * (j < ns ? (T)Q[(long long)c * ns + j] : T(0));
        out[(long long)c * ldo + x] = t;
    }
}

template <typename T>
static void launch_rotate_small(const T *Y, long long ldy, const double *Q, T *out, long long ldo, long long nd, int ns,
                                hipStream_t s)
{
    const dim3 g((unsigned)((nd + 255) / 256)), b(256);
    if (ns <= 4)
        hipLaunchKernelGGL((rotate_small_kernel<T, 4>), g, b, 0, s, Y, ldy, Q, out, ldo, nd, ns);
    else if (ns <= 8)
        hipLaunchKernelGGL((rotate_small_kernel<T, 8>), g, b, 0, s, Y, ldy, Q, out, ldo, nd, ns);
    else
        hipLaunchKernelGGL((rotate_small_kernel<T, 16>), g, b, 0, s, Y, ldy, Q, out, ldo, nd, ns);
}

// ---------------------------------------------------------------- BLAS handles

// rocBLAS handles are not safe for concurrent use, and a handle's device
// workspace stays in use until the work enqueued with it has run.  Each call
// leases a handle from a per-device pool: one last used on the same stream
// (stream order protects its workspace) or one whose completion event has
// fired; otherwise a new handle is made.  Returning a lease records the event
// on the call's stream.  Handles are kept until the process ends, except one
// that a call was thrown out of: its state is unknown, it is left behind.
namespace {
struct PooledBlas {
    rocblas_handle h = nullptr;
    hipEvent_t done = nullptr;
    hipStream_t last = nullptr;
};
std::mutex g_blas_mu;
std::map<int, std::vector<PooledBlas>> g_blas_free;

struct BlasLease {
    int dev = 0;
    hipStream_t stream;
    PooledBlas e;
    rocblas_handle h = nullptr;
    bool thrown = false;
    explicit BlasLease(hipStream_t s) : stream(s)
    {
        (void)hipGetDevice(&dev);
        bool found = false;
        {
            std::lock_guard<std::mutex> lk(g_blas_mu);
            auto &v = g_blas_free[dev];
            for (size_t i = 0; i < v.size(); ++i) {
                bool idle = v[i].last == s;
                if (!idle) {
                    const hipError_t q = hipEventQuery(v[i].done);
                    idle = q == hipSuccess;
                    // a pending event is the expected answer, not an error of
                    // this thread's later calls
                    if (q == hipErrorNotReady) (void)hipGetLastError();
                }
                if (idle) {
                    e = v[i];
                    v.erase(v.begin() + (long)i);
                    found = true;
                    break;
                }
            }
        }
        if (!found) {
            // handles are created one at a time (creation is not documented as thread-safe)
            std::lock_guard<std::mutex> lk(g_blas_mu);
            if (rocblas_create_handle(&e.h) != rocblas_status_success) {
                e.h = nullptr;
                return;
            }
            if (hipEventCreateWithFlags(&e.done, hipEventDisableTiming) != hipSuccess) {
                rocblas_destroy_handle(e.h);
                e.h = nullptr;
                return;
            }
            // no atomics: results must not depend on scheduling
            rocblas_set_atomics_mode(e.h, rocblas_atomics_not_allowed);
        }
        rocblas_set_stream(e.h, s);
        h = e.h;
    }
    ~BlasLease()
    {
        if (!h || thrown) return;
        quiet([&] {
            (void)hipEventRecord(e.done, stream);
            e.last = stream;
            std::lock_guard<std::mutex> lk(g_blas_mu);
            g_blas_free[dev].push_back(e);
        });
    }
    BlasLease(const BlasLease &) = delete;
    BlasLease &operator=(const BlasLease &) = delete;

    // One library call, its status in rs.  The libraries are C++ inside and do
    // not all catch their own exceptions (std::bad_variant_access has been seen
    // to leave one): they end here, with the call, not in the caller's thread.
    template <typename F>
    int call(const char *what, rocblas_status &rs, F &&f)
    {
        try {
            rs = f();
            return SPARC_OK;
        } catch (const std::exception &x) {
            thrown = true;
            (void)hipGetLastError();
            return fail(SPARC_E_HIP, std::string(what) + " threw: " + x.what());
        } catch (...) {
            thrown = true;
            (void)hipGetLastError();
            return fail(SPARC_E_HIP, std::string(what) + " threw an unknown exception");
        }
    }
};
// A HIP error state left behind by a library call that itself reported
// success.  The one code seen so far (hipErrorStreamCaptureUnsupported, after
// rocSOLVER's generalized eigensolver on worker threads that capture nothing)
// is cleared and
// counted, with its first occurrences written to stderr; any other code fails
// the call.
std::atomic<long long> g_cleared_errors{0};

int note_library_error(const char *call, hipError_t e)
{
    if (e != hipErrorStreamCaptureUnsupported)
        return fail(SPARC_E_HIP, std::string(call) + " returned success but left HIP error: " + hipGetErrorString(e));
    const long long n = ++g_cleared_errors;
    if (n <= 8)
        fprintf(stderr, "sparc: cleared HIP error left by %s after success (%s), occurrence %lld\n", call,
                hipGetErrorString(e), n);
    return SPARC_OK;
}
}  // namespace

// ---------------------------------------------------------------- tridiagonal eigenvalues

// number of eigenvalues of the symmetric tridiagonal (alpha, beta) below x
static int sturm_count(const double *alpha, const double *beta, int k, double x)
{
    int count = 0;
    double q = 1.0;
    for (int i = 0; i < k; ++i) {
        const double b2 = i > 0 ? beta[i - 1] * beta[i - 1] : 0.0;
        q = (alpha[i] - x) - (i > 0 ? b2 / q : 0.0);
        if (q == 0.0) q = -1e-300;
        if (q < 0) ++count;
    }
    return count;
}

static void tridiag_eigenvalues(const double *alpha, const double *beta, int k, double *theta)
{
    double lo = INFINITY, hi = -INFINITY;
    for (int i = 0; i < k; ++i) {
        const double r = (i > 0 ? std::fabs(beta[i - 1]) : 0.0) + (i + 1 < k ? std::fabs(beta[i]) : 0.0);
        lo = std::min(lo, alpha[i] - r);
        hi = std::max(hi, alpha[i] + r);
    }
    const double pad = 1e-12 * std::max(1.0, std::max(std::fabs(lo), std::fabs(hi)));
    lo -= pad;
    hi += pad;
    for (int j = 0; j < k; ++j) {
        // the (j+1)-th smallest eigenvalue: smallest x with count(x) > j
        double a = lo, b = hi;
        for (int it = 0; it < 200; ++it) {
            const double mid = 0.5 * (a + b);
            if (mid <= a || mid >= b) break;
            if (sturm_count(alpha, beta, k, mid) > j)
                b = mid;
            else
                a = mid;
        }
        theta[j] = 0.5 * (a + b);
    }
}

}  // namespace sparc

using namespace sparc;

extern "C" {

size_t sparc_lanczos_workspace_bytes(const sparc_op *op, int32_t k)
{
    if (!op || k < 1) return 0;
    size_t b = align_up((size_t)op->nd * (k + 1) * sizeof(double));  // vectors u_0..u_{k-1} and one more
    b += gather_bytes(op, SPARC_F64, 1);                                  // gathered projections
    b += align_up((size_t)(4 * k + 8) * sizeof(double));                  // alpha, nu
    b += align_up((size_t)kRedBlocks * (k + 3) * sizeof(double));         // partials: inner products, |w|^2 twice
    b += align_up((size_t)lanczos_dot_blocks(op) * sizeof(double));        // u^T H_loc u partials
    b += align_up((size_t)(3 * (k + 2) + k + 1) * sizeof(double));        // omega rows, ||T|| per step
    b += align_up((size_t)(2 * k + 1) * sizeof(int));                       // reorthogonalisation flags per step
    return b;
}

// Lanczos with partial re-orthogonalisation: w = H v_j, alpha_j = v_j^T H v_j,
// w -= alpha_j v_j + beta_{j-1} v_{j-1}, beta_j = |w|; when the omega
// recurrence (omega_dots_kernel) estimates a loss of orthogonality beyond sqrt(eps),
// one classical Gram-Schmidt pass against v_0 .. v_j (c = V^T w, w -= V c) and
// a new beta_j; v_{j+1} = w / beta_j.  Every step is enqueued without a host
// round trip: the conditional pass reads its flag on the device.
int sparc_lanczos(const sparc_op *op, int32_t k, const double *v0, double *alpha, double *beta, double *theta,
                  void *ws, size_t ws_bytes, void *stream)
{
    if (!op || !v0 || !theta) return fail(SPARC_E_ARG, "null argument");
    if (k < 1 || k > op->nd) return fail(SPARC_E_ARG, "need 1 <= k <= N_d");
    const size_t need = sparc_lanczos_workspace_bytes(op, k);
    if (!ws || ws_bytes < need) return fail(SPARC_E_WORKSPACE, "workspace too small");
    TraceRange trace("sparc_lanczos");
    hipStream_t s = (hipStream_t)stream;
    const long long n = op->nd;
    char *p = (char *)ws;
    double *V = (double *)p;  // k+1 vectors of n
    p += align_up((size_t)n * (k + 1) * sizeof(double));
    double *G = (double *)p;
    p += gather_bytes(op, SPARC_F64, 1);
    double *d_alpha = (double *)p;
    double *d_nu = d_alpha + k;  // k + 1 entries; beta_j = nu_{j+1}
    p += align_up((size_t)(4 * k + 8) * sizeof(double));
    double *partial = (double *)p;  // inner products (kDotBlocks per vector)
    double *npart[2];               // |w|^2, one per block, by the parity of the step
    npart[0] = partial + (size_t)kDotBlocks * (k + 1);
    npart[1] = npart[0] + kRedBlocks;
    p += align_up((size_t)kRedBlocks * (k + 3) * sizeof(double));
    double *dotp = (double *)p;  // step kernel partials of u_j^T H_loc u_j
    const int ndot = (int)lanczos_dot_blocks(op);
    p += align_up((size_t)ndot * sizeof(double));
    double *rows = (double *)p;  // three rows of orthogonality estimates, k + 2 entries each
    double *d_anorm = rows + 3 * (k + 2);  // ||T|| estimate after each step (k + 1)
    p += align_up((size_t)(3 * (k + 2) + k + 1) * sizeof(double));
    int *d_owed = (int *)p;     // k + 1: orthogonalise the vector of step j regardless
    int *d_full = d_owed + k + 1;  // k: the vector of step j is orthogonalised
    const double eps1 = 0.5 * std::sqrt((double)n) * 2.220446049250313e-16;

    const dim3 rg(kRedBlocks), tb(256);
    int st;
    hipLaunchKernelGGL(omega_init, dim3(1), tb, 0, s, rows, k + 2, d_owed, d_anorm, d_nu);
    // u_0 = v0 / |v0|
    hipLaunchKernelGGL(norm2_kernel, rg, tb, 0, s, v0, n, npart[1]);
    hipLaunchKernelGGL(scale_by_norm, rg, tb, 0, s, V, v0, (const double *)npart[1], n);
    const int nproj = op->nproj_total;
    const bool fused = op->natoms > 0 && nproj <= kLanczosProj;
    const LanczosScatter sc{op->d_nl_seg, op->d_nl_pts, op->d_nl_off, (const int4 *)op->d_nl_ent, op->d_nl_proj,
                            op->d_chi64};
    for (int j = 0; j < k; ++j) {
        double *uj = V + (long long)j * n, *w = uj + n;
        // w = H_loc u_j, with the two parts of u_j^T H u_j left as partials
        if ((st = launch_lanczos_h_f64(op, uj, w, dotp, G, s))) return st;
        const LanczosAlpha q{dotp, ndot, G, op->d_hg64, nproj, j > 0 ? d_full + j - 1 : nullptr, npart[(j + 1) & 1]};
        if (j + 1 == k) {
            hipLaunchKernelGGL(alpha_finish, dim3(1), tb, 0, s, q, d_nu + j, d_alpha + j);
            break;
        }
        // w += V_nl u_j; alpha_j; w / nu_j - alpha_j v_j - beta_{j-1} v_{j-1}; partials of |w|^2
        const double *ujm = j > 0 ? uj - n : nullptr;
        if (fused) {
            hipLaunchKernelGGL(lanczos_3term<true>, rg, tb, 0, s, w, (const double *)uj, ujm, q, sc, d_nu + j,
                               d_alpha + j, n, npart[j & 1]);
        } else {
            if ((st = launch_scatter(op, SPARC_F64, w, n, 1, G, kGatherSplit, 1.0, s))) return st;
            hipLaunchKernelGGL(lanczos_3term<false>, rg, tb, 0, s, w, (const double *)uj, ujm, q, sc, d_nu + j,
                               d_alpha + j, n, npart[j & 1]);
        }
        // beta_j, the orthogonality estimates and, when they ask for it, one
        // classical Gram-Schmidt pass against v_0 .. v_j, whose new |w|^2
        // partials the next step finishes into beta_j
        const double *Wc = rows + (size_t)(j % 3) * (k + 2);
        const double *Wp = rows + (size_t)((j + 2) % 3) * (k + 2);
        double *Wn = rows + (size_t)((j + 1) % 3) * (k + 2);
        const int nv = j + 1;
        hipLaunchKernelGGL(omega_dots_kernel, rg, tb, 0, s, (const double *)d_alpha, d_nu + 1, j, eps1, Wp, Wc, Wn,
                           d_owed, d_full, d_anorm, (const double *)npart[j & 1], (const double *)V, (long long)n,
                           (const double *)w, n, partial);
        hipLaunchKernelGGL(orth_apply_norm, rg, tb, 0, s, w, (const double *)V, (long long)n, nv,
                           (const double *)partial, (const double *)d_nu, n, npart[j & 1], (const int *)(d_full + j));
        SPARC_HIP(hipGetLastError());
    }
    SPARC_HIP(hipGetLastError());
    std::vector<double> ha(k), hb(std::max(1, k - 1));
    SPARC_HIP(hipMemcpyAsync(ha.data(), d_alpha, k * sizeof(double), hipMemcpyDeviceToHost, s));
    if (k > 1) SPARC_HIP(hipMemcpyAsync(hb.data(), d_nu + 1, (k - 1) * sizeof(double), hipMemcpyDeviceToHost, s));
    SPARC_HIP(hipStreamSynchronize(s));
    for (int j = 0; j + 1 < k; ++j)
        if (!(hb[j] > 0.0) || !std::isfinite(hb[j])) return fail(SPARC_E_BREAKDOWN, "Lanczos breakdown at step " + std::to_string(j));
    for (int j = 0; j < k; ++j)
        if (!std::isfinite(ha[j])) return fail(SPARC_E_BREAKDOWN, "non-finite Lanczos coefficient");
    tridiag_eigenvalues(ha.data(), hb.data(), k, theta);
    if (alpha) std::copy(ha.begin(), ha.end(), alpha);
    if (beta && k > 1) std::copy(hb.begin(), hb.begin() + (k - 1), beta);
    return SPARC_OK;
}

// points per chunk for about nch chunks: a multiple of the staged slice
static long long rr_points(long long nd, long long nch)
{
    nch = std::max<long long>(1, std::min<long long>(nch, nd / kRrK));
    const long long c = ((nd + nch - 1) / nch + kRrK - 1) / kRrK * kRrK;
    return std::max<long long>(c, kRrK);
}

// ns x ns pairs of partial matrices the workspace has room for
static long long rr_room(long long nd, int ns)
{
    const long long nt = (ns + kRrTile - 1) / kRrTile;
    const long long tiles = nt * (nt + 1) / 2;
    const long long c = rr_points(nd, std::max<long long>(64, (512 + tiles - 1) / tiles));
    return (nd + c - 1) / c;
}

// The chip holds 768 workgroups of the projection (three per CU): as many
// chunks as make whole multiples of that and whose packed triangles fit the
// room.  160^3 x 100: 768 workgroups 6.82 ms, 512 6.99, 640 7.28 (the whole
// step); 160^3 x 600: 125 chunks (8.95 times 768) 83.2 ms, 64 chunks 84.9.
static long long rr_chunk(long long nd, int ns)
{
    const long long nt = (ns + kRrTile - 1) / kRrTile;
    const long long tiles = nt * (nt + 1) / 2;
    const long long most = std::max<long long>(1, rr_room(nd, ns) * 2 * ns / (ns + 1));
    const long long rounds = most * tiles / 768;
    return rr_points(nd, rounds > 0 ? 768 * rounds / tiles : most);
}

size_t sparc_rr_workspace_bytes(const sparc_op *op, int32_t dtype, int32_t ns)
{
    if (!op || ns < 1) return 0;
    size_t b = 0;
    b += align_up((size_t)op->nd * ns * sizeof(double));                           // H Y
    b += gather_bytes(op, SPARC_F64, ns);                                           // gathered projections
    b += 2 * align_up((size_t)ns * ns * sizeof(double));                           // H_s, M_s
    b += align_up(((size_t)ns + 1) * sizeof(double)) + align_up((size_t)ns * sizeof(double));  // D and info, E
    b += align_up((size_t)rr_room(op->nd, ns) * 2 * ns * ns * sizeof(double));     // projection partials
    return b;
}

int sparc_rayleigh_ritz(const sparc_op *op, int32_t dtype, const void *Y, int64_t ldy, int32_t ns, double *theta,
                        double *evec, void *ws, size_t ws_bytes, void *stream)
{
    g_rr_rank_deficient = false;
    if (!op || !Y || !theta) return fail(SPARC_E_ARG, "null argument");
    if (dtype != SPARC_F64 && dtype != SPARC_F32) return fail(SPARC_E_ARG, "bad dtype");
    if (ns < 1 || ldy < op->nd) return fail(SPARC_E_SHAPE, "ns < 1 or ldy < N_d");
    if ((long long)8 * ldy + op->nd >= (1LL << 32))
        return fail(SPARC_E_SHAPE, "ldy too large for the projection kernel");
    const size_t need = sparc_rr_workspace_bytes(op, dtype, ns);
    if (!ws || ws_bytes < need) return fail(SPARC_E_WORKSPACE, "workspace too small");
    TraceRange trace("sparc_rayleigh_ritz");
    hipStream_t s = (hipStream_t)stream;
    const long long nd = op->nd;
    char *p = (char *)ws;
    double *HY = (double *)p;
    p += align_up((size_t)nd * ns * sizeof(double));
    double *G = (double *)p;
    p += gather_bytes(op, SPARC_F64, ns);
    double *Hs = (double *)p;
    p += align_up((size_t)ns * ns * sizeof(double));
    double *Ms = (double *)p;
    p += align_up((size_t)ns * ns * sizeof(double));
    double *D = (double *)p;  // ns values, then the solver's status
    int *info = (int *)(D + ns);
    p += align_up(((size_t)ns + 1) * sizeof(double));
    double *E = (double *)p;
    p += align_up((size_t)ns * sizeof(double));
    double *partial = (double *)p;

    int st;
    StepLaunch L = choose_step_launch(op, SPARC_F64, ns);
    StepCoef hc{1.0, 0.0, 0.0, 0};
    const long long kc = rr_chunk(nd, ns);
    const int nch = (int)((nd + kc - 1) / kc);
    const int nt = (ns + kRrTile - 1) / kRrTile;
    const dim3 pg((unsigned)(nch * (nt * (nt + 1) / 2)), 1, 1);
    if (dtype == SPARC_F64) {
        const FLaunch V = choose_vec_launch(op, SPARC_F64, ns, {ldy, nd});
        if ((st = launch_h_step(op, SPARC_F64, Y, ldy, nullptr, 0, HY, nd, ns, G, hc, L, s, &V))) return st;
        hipLaunchKernelGGL(rr_project_kernel<double>, pg, dim3(256), 0, s, (const double *)Y, (long long)ldy,
                           (const double *)HY, nd, nd, ns, kc, partial);
    } else {
        // H in FP64 on the FP32 values, widened as they are loaded
        const float *Yf = (const float *)Y;
        const int nparts = op->natoms > 0 && gather_wide(op, ns) ? 1 : kGatherSplit;
        if ((st = launch_gather_f32_to_f64(op, Yf, ldy, ns, G, nparts, s))) return st;
        if ((st = launch_step_f32_to_f64(op, Yf, ldy, HY, nd, ns, hc, choose_mixed_launch(op, ns), s))) return st;
        if ((st = launch_scatter(op, SPARC_F64, HY, nd, ns, G, nparts, 1.0, s))) return st;
        hipLaunchKernelGGL(rr_project_kernel<float>, pg, dim3(256), 0, s, Yf, (long long)ldy, (const double *)HY, nd,
                           nd, ns, kc, partial);
    }
    const long long tot = (long long)ns * (ns + 1);
    if (ns <= 64)
        hipLaunchKernelGGL(rr_reduce_kernel<16>, dim3((unsigned)((tot + 15) / 16)), dim3(256), 0, s, partial, nch, ns, Ms,
                           Hs);
    else
        hipLaunchKernelGGL(rr_reduce_kernel<1>, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, partial, nch, ns,
                           Ms, Hs);
    SPARC_HIP(hipGetLastError());

    if (ns <= 64) {
        // one-workgroup Cholesky + Jacobi
        if ((st = launch_small_sygv(Hs, Ms, ns, D, evec ? evec : Hs, info, s))) return st;
    } else {
        BlasLease lease(s);
        rocblas_handle hb = lease.h;
        if (!hb) return fail(SPARC_E_HIP, "rocblas_create_handle failed");
        // anything still pending here was left by an earlier call of this thread
        const hipError_t before = hipGetLastError();
        if (before != hipSuccess)
            return fail(SPARC_E_HIP, std::string("HIP error pending before the eigensolver: ") + hipGetErrorString(before));
        // M_s = U^T U (rocSOLVER Cholesky); the reduction to the standard
        // problem C = U^-T H_s U^-1 and the back-transformation q = U^-1 z by
        // blocked triangular solves (rocBLAS trsm); C z = theta z by rocSOLVER's
        // divide-and-conquer symmetric eigensolver.  (rocsolver_dsygvd's own
        // reduction issues ~600 matrix-vector solves per call at N_s = 600.)
        auto lib_call = [&](const char *what, auto &&f) -> int {
            rocblas_status rs;
            if (int threw = lease.call(what, rs, f)) return threw;
            const hipError_t after = hipGetLastError();
            if (rs != rocblas_status_success)
                return fail(SPARC_E_HIP, std::string(what) + " failed: " + rocblas_status_to_string(rs) +
                                             (after != hipSuccess ? std::string(", HIP: ") + hipGetErrorString(after) : ""));
            if (after != hipSuccess) return note_library_error(what, after);
            return SPARC_OK;
        };
        if ((st = lib_call("rocsolver_dpotrf", [&] { return rocsolver_dpotrf(hb, rocblas_fill_upper, ns, Ms, ns, info); })))
            return st;
        int pinfo = 0;
        SPARC_HIP(hipMemcpyAsync(&pinfo, info, sizeof(int), hipMemcpyDeviceToHost, s));
        SPARC_HIP(hipStreamSynchronize(s));
        if (pinfo != 0) {
            g_rr_rank_deficient = true;
            return fail(SPARC_E_BREAKDOWN, "Cholesky of M_s failed (info=" + std::to_string(pinfo) +
                                               "): the filtered block is numerically rank deficient");
        }
        // Hs = op(U)^-1 Hs (left) or Hs op(U)^-1 (right)
        auto solve = [&](rocblas_side side, rocblas_operation op_u) -> int {
            const double one = 1.0;
            return lib_call("rocblas_dtrsm", [&] {
                return rocblas_dtrsm(hb, side, rocblas_fill_upper, op_u, rocblas_diagonal_non_unit, ns, ns, &one, Ms, ns,
                                     Hs, ns);
            });
        };
        if ((st = solve(rocblas_side_left, rocblas_operation_transpose))) return st;
        if ((st = solve(rocblas_side_right, rocblas_operation_none))) return st;
        if ((st = lib_call("rocsolver_dsyevd", [&] {
                 return rocsolver_dsyevd(hb, evec ? rocblas_evect_original : rocblas_evect_none, rocblas_fill_upper, ns,
                                         Hs, ns, D, E, info);
             })))
            return st;
        if (evec && (st = solve(rocblas_side_left, rocblas_operation_none))) return st;
    }
    // Ritz values and the solver's status in one copy
    std::vector<double> host((size_t)ns + 1);
    SPARC_HIP(hipMemcpyAsync(host.data(), D, ((size_t)ns + 1) * sizeof(double), hipMemcpyDeviceToHost, s));
    if (evec && ns > 64)
        SPARC_HIP(hipMemcpyAsync(evec, Hs, (size_t)ns * ns * sizeof(double), hipMemcpyDeviceToDevice, s));
    SPARC_HIP(hipStreamSynchronize(s));
    std::copy(host.begin(), host.begin() + ns, theta);
    int hinfo;
    std::memcpy(&hinfo, &host[ns], sizeof(int));
    if (hinfo != 0) {
        if (ns <= 64 && hinfo == ns + 1)
            return fail(SPARC_E_BREAKDOWN, "Jacobi eigensolver did not converge within its sweep limit");
        if (ns > 64)
            return fail(SPARC_E_BREAKDOWN, "rocsolver_dsyevd: the tridiagonal eigensolver did not converge (info=" +
                                               std::to_string(hinfo) + ")");
        // the small solver's Cholesky factorisation of M_s failed (info = the
        // failing column)
        g_rr_rank_deficient = true;
        return fail(SPARC_E_BREAKDOWN, "Cholesky of M_s failed (info=" + std::to_string(hinfo) +
                                           "): the filtered block is numerically rank deficient");
    }
    return SPARC_OK;
}

int64_t sparc_cleared_hip_errors(void) { return g_cleared_errors.load(); }

size_t sparc_rotate_workspace_bytes(int32_t dtype, int32_t ns)
{
    if (ns < 1) return 0;
    if (dtype == SPARC_F64) return (size_t)rot_ldq(ns) * rot_ncols<double>(ns) * sizeof(double);
    if (dtype == SPARC_F32) return (size_t)rot_ldq(ns) * rot_ncols<float>(ns) * sizeof(float);
    return 0;
}

int sparc_rotate(int32_t dtype, const void *Y, int64_t ldy, int64_t nd, int32_t ns, const double *Q, void *out,
                 int64_t ldo, void *ws, size_t ws_bytes, void *stream)
{
    if (!Y || !Q || !out) return fail(SPARC_E_ARG, "null argument");
    if (dtype != SPARC_F64 && dtype != SPARC_F32) return fail(SPARC_E_ARG, "bad dtype");
    if (ns < 1 || nd < 1 || ldy < nd || ldo < nd) return fail(SPARC_E_SHAPE, "bad shape");
    const size_t es = elem_size(dtype);
    const size_t by = (size_t)((ns - 1) * ldy + nd) * es, bo = (size_t)((ns - 1) * ldo + nd) * es;
    const char *pa = (const char *)Y, *pb = (const char *)out;
    if (pa < pb + bo && pb < pa + by) return fail(SPARC_E_ALIAS, "Y and out overlap");
    const size_t need = sparc_rotate_workspace_bytes(dtype, ns);
    if (!ws || ws_bytes < need) return fail(SPARC_E_WORKSPACE, "workspace too small");
    const char *pw = (const char *)ws;
    if ((pw < pa + by && pa < pw + need) || (pw < pb + bo && pb < pw + need))
        return fail(SPARC_E_ALIAS, "workspace overlaps Y or out");
    TraceRange trace("sparc_rotate");
    hipStream_t s = (hipStream_t)stream;
    if (launch_rotate_mfma(dtype, Y, ldy, Q, out, ldo, nd, ns, s)) {
        SPARC_HIP(hipGetLastError());
        return SPARC_OK;
    }
    const unsigned gx = (unsigned)((nd + 255) / 256);
    const int ldq = rot_ldq(ns);
    // Blocks wider than one column block of the kernel below would re-read Y
    // once per block of output columns; the product is then a plain GEMM on
    // the matrix cores (rocBLAS, atomics off: deterministic).
    const bool gemm = ns > (dtype == SPARC_F64 ? RotTile<double>::cols : RotTile<float>::cols) &&
                      nd <= 0x7fffffffLL && ldy <= 0x7fffffffLL && ldo <= 0x7fffffffLL;
    if (gemm) {
        BlasLease lease(s);
        if (!lease.h) return fail(SPARC_E_HIP, "rocblas_create_handle failed");
        rocblas_status rs;
        int st;
        if (dtype == SPARC_F64) {
            hipLaunchKernelGGL(pad_rotation<double>, stream_grid((long long)ldq * ns), dim3(256), 0, s, Q, ns,
                               (double *)ws, ldq, ns);
            const double one = 1.0, zero = 0.0;
            st = lease.call("rocblas_dgemm", rs, [&] {
                return rocblas_dgemm(lease.h, rocblas_operation_none, rocblas_operation_none, (rocblas_int)nd, ns, ns, &one,
                                     (const double *)Y, (rocblas_int)ldy, (const double *)ws, ldq, &zero, (double *)out,
                                     (rocblas_int)ldo);
            });
        } else {
            hipLaunchKernelGGL(pad_rotation<float>, stream_grid((long long)ldq * ns), dim3(256), 0, s, Q, ns,
                               (float *)ws, ldq, ns);
            const float one = 1.0f, zero = 0.0f;
            st = lease.call("rocblas_sgemm", rs, [&] {
                return rocblas_sgemm(lease.h, rocblas_operation_none, rocblas_operation_none, (rocblas_int)nd, ns, ns, &one,
                                     (const float *)Y, (rocblas_int)ldy, (const float *)ws, ldq, &zero, (float *)out,
                                     (rocblas_int)ldo);
            });
        }
        if (st) return st;
        const hipError_t after = hipGetLastError();
        if (rs != rocblas_status_success)
            return fail(SPARC_E_HIP, std::string("rocBLAS GEMM of the rotation failed: ") + rocblas_status_to_string(rs));
        if (after != hipSuccess) return fail(SPARC_E_HIP, std::string("rotation: ") + hipGetErrorString(after));
        return SPARC_OK;
    }
    if (ns <= kRotSmall) {
        if (dtype == SPARC_F64)
            launch_rotate_small((const double *)Y, ldy, Q, (double *)out, ldo, nd, ns, s);
        else
            launch_rotate_small((const float *)Y, ldy, Q, (float *)out, ldo, nd, ns, s);
        SPARC_HIP(hipGetLastError());
        return SPARC_OK;
    }
    if (dtype == SPARC_F64) {
        const int ncp = rot_ncols<double>(ns);
        hipLaunchKernelGGL(pad_rotation<double>, stream_grid((long long)ldq * ncp), dim3(256), 0, s, Q, ns,
                           (double *)ws, ldq, ncp);
        hipLaunchKernelGGL(rotate_kernel<double>, dim3(gx, ncp / RotTile<double>::cols), dim3(256), 0, s,
                           (const double *)Y, (long long)ldy, (const double *)ws, ldq, (double *)out, (long long)ldo,
                           (long long)nd, ns);
    } else {
        const int ncp = rot_ncols<float>(ns);
        hipLaunchKernelGGL(pad_rotation<float>, stream_grid((long long)ldq * ncp), dim3(256), 0, s, Q, ns,
                           (float *)ws, ldq, ncp);
        hipLaunchKernelGGL(rotate_kernel<float>, dim3(gx, ncp / RotTile<float>::cols), dim3(256), 0, s,
                           (const float *)Y, (long long)ldy, (const float *)ws, ldq, (float *)out, (long long)ldo,
                           (long long)nd, ns);
    }
    SPARC_HIP(hipGetLastError());
    return SPARC_OK;
}

}  // extern "C"
