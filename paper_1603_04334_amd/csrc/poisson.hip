// Electrostatic potential (Sec. 3.3): -(1/4 pi) lap_h phi = c - d on the grid
// with zero Dirichlet padding (Eq. FD:PoissonDiscrete), c = rho + b the total
// charge and d the charge correction of Eq. Phi:correction, which carries the
// values of phi just outside the grid from the multipole expansion of c to
// l_max (Eq. phi:BC:discrete and the discrete moments Q_lm that follow it).
// Solved by conjugate gradients with a block-Jacobi preconditioner (Sec. 4).
//
// Layout and kernels (everything FP64, on the device):
//  * moments: one pass over the grid, each thread accumulating all
//    (l_max+1)^2 products r^l Y_lm c (regular solid harmonics from their
//    Cartesian recurrences, expansion centre = domain centre); one partial
//    per workgroup, summed in a fixed order;
//  * boundary values of phi on the six off-grid slabs n_o nodes deep (only
//    nodes one axis step off a face are ever read by the stencil);
//  * right-hand side c - d, with d from the slabs, and the partial sums of
//    its square;
//  * CG iteration, three launches: q = A p with the partial sums of p.q (the
//    stencil kernel of vstep.hip on vectors without a potential; A =
//    (1/2 pi) (-1/2 lap_h)); r -= alpha q, z = M^-1 r per block and the
//    partials of r.z and r.r; x += alpha p, the convergence test and
//    p = z + beta p.  Scalars never leave the device: every workgroup finishes
//    the partial sums it needs in the same fixed order, so alpha, beta and the
//    convergence test are bitwise the same everywhere.  The host enqueues
//    iterations in chunks and reads one flag per chunk; kernels of iterations
//    after the converged one return at once.
//  * block Jacobi, each block's operator inverted exactly: blocks of 4 x 4 x 4
//    nodes in the eigenbasis of their axes (bj_diag_kernel), other block shapes
//    by a dense symmetric inverse per shape, in bricks along z so that global
//    accesses are coalesced rows (bj_kernel).
//  What bounds it: 11 passes of 8 N_d bytes per iteration (14 with p.q and the
//  x update in passes of their own): 160^3 138 -> 77 us per iteration, 361 MB at
//  4.7 TB/s; 96^3 57 -> 30 us; 49 x 44 x 41 33 -> 27 us, launches and their
//  latency.
#include <algorithm>
#include <cmath>
#include <vector>

#include "internal.hpp"

namespace sparc {
namespace {

constexpr int kLmax = 6;                           // largest expansion order supported
constexpr int kNM = (kLmax + 1) * (kLmax + 1);     // moments
constexpr int kPT = 256;                           // threads per workgroup
constexpr int kBjStage = 64;                       // largest block (nodes) whose inverse is staged in LDS
constexpr int kRedMax = 1024;                      // workgroups of the reduction kernels
// CG iterations enqueued between convergence reads.  A read leaves the chip idle
// for about 30 us, an iteration after the converged one costs three empty
// launches.  From zero 24 (8, 16, 24, 32: 24^3 1.68, 1.62, 1.43, 1.72 ms; 96^3
// 7.56, 7.06, 6.90, 6.90 ms; 160^3 30.8, 29.9, 29.6, 29.5 ms; a small grid's time
// also depends on where its last iteration falls in a chunk).  A solve from a good
// guess may need few: twice half a chunk first.
constexpr int kChunk = 24;
inline int chunk_from(int it, bool guess) { return guess && it < kChunk ? kChunk / 2 : kChunk; }
constexpr double kFourPi = 12.566370614359172954;  // 4 pi

struct HarmNorm {
    double c[kNM];
};

// device-side state: the iteration that reached the tolerance (-1: the start,
// kNotDone: none yet), and the scalars handed from launch to launch, one slot
// per parity of the iteration (a launch reads the slot of its own iteration and
// writes the other's)
constexpr int kNotDone = 0x7fffffff;
struct PcgState {
    int done;
    int iters;
    double rr, bb;
    double rz[2];  // r.z at the start of an iteration
    double alpha;
};

// regular solid harmonics R_lm(x) = |x|^l Y_lm(x/|x|), index l*l + l + m:
// (x + i y)^m = C_m + i S_m, the polynomial P_l^m(z, r^2) of the associated
// Legendre recurrence in l, and R_lm = N_lm P_l^m C_m (m >= 0),
// R_l,-m = N_lm P_l^m S_m
__device__ __forceinline__ void solid_harmonics(double x, double y, double z, const HarmNorm &nrm, double (&R)[kNM])
{
    const double r2 = x * x + y * y + z * z;
    double C[kLmax + 1], S[kLmax + 1];
    C[0] = 1.0;
    S[0] = 0.0;
#pragma unroll
    for (int m = 1; m <= kLmax; ++m) {
        C[m] = x * C[m - 1] - y * S[m - 1];
        S[m] = x * S[m - 1] + y * C[m - 1];
    }
    double dfact = 1.0;  // (2m - 1)!!
#pragma unroll
    for (int m = 0; m <= kLmax; ++m) {
        if (m > 0) dfact *= (2 * m - 1);
        double p2 = dfact, p1 = 0.0;
#pragma unroll
        for (int l = m; l <= kLmax; ++l) {
            double P;
            if (l == m) {
                P = p2;
            } else if (l == m + 1) {
                P = (2 * m + 1) * z * p2;
                p1 = P;
            } else {
                P = ((2 * l - 1) * z * p1 - (l + m - 1) * r2 * p2) / (l - m);
                p2 = p1;
                p1 = P;
            }
            R[l * l + l + m] = nrm.c[l * l + l + m] * P * C[m];
            if (m > 0) R[l * l + l - m] = nrm.c[l * l + l - m] * P * S[m];
        }
    }
}

__device__ __forceinline__ double wave_sum(double v)
{
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// sum over the 256 threads, the same value in every thread (fixed order)
__device__ __forceinline__ double block_sum(double v, double *red)
{
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return (red[0] + red[1]) + (red[2] + red[3]);
}

// sum of n partials in a fixed order, the same value in every thread
__device__ __forceinline__ double sum_partials(const double *part, int n, double *red)
{
    double v = 0.0;
    for (int i = threadIdx.x; i < n; i += kPT) v += part[i];
    return block_sum(v, red);
}

// two such sums with one pair of barriers
__device__ __forceinline__ void sum_partials2(const double *a, const double *b, int n, double (&red)[8], double &sa,
                                              double &sb)
{
    double v = 0.0, w = 0.0;
    for (int i = threadIdx.x; i < n; i += kPT) {
        v += a[i];
        w += b[i];
    }
    v = wave_sum(v);
    w = wave_sum(w);
    if ((threadIdx.x & 63) == 0) {
        red[threadIdx.x >> 6] = v;
        red[4 + (threadIdx.x >> 6)] = w;
    }
    __syncthreads();
    sa = (red[0] + red[1]) + (red[2] + red[3]);
    sb = (red[4] + red[5]) + (red[6] + red[7]);
}

struct GridGeo {
    int n0, n1, n2;
    long long nd;
    double h;
    double c0, c1, c2;  // domain centre
};

__device__ __forceinline__ void node_pos(const GridGeo &g, long long t, int &i, int &j, int &k, double &x, double &y,
                                         double &z)
{
    k = (int)(t % g.n2);
    const long long u = t / g.n2;
    j = (int)(u % g.n1);
    i = (int)(u / g.n1);
    x = (i + 1) * g.h - g.c0;
    y = (j + 1) * g.h - g.c1;
    z = (k + 1) * g.h - g.c2;
}

__global__ void __launch_bounds__(kPT) moments_kernel(const double *__restrict__ charge, const GridGeo g,
                                                      const HarmNorm nrm, double *__restrict__ partial)
{
    double acc[kNM];
#pragma unroll
    for (int q = 0; q < kNM; ++q) acc[q] = 0.0;
    for (long long t = blockIdx.x * (long long)kPT + threadIdx.x; t < g.nd; t += (long long)gridDim.x * kPT) {
        const double f = charge[t];
        int i, j, k;
        double x, y, z;
        node_pos(g, t, i, j, k, x, y, z);
        double R[kNM];
        solid_harmonics(x, y, z, nrm, R);
#pragma unroll
        for (int q = 0; q < kNM; ++q) acc[q] += R[q] * f;
    }
    __shared__ double red[4][kNM];
#pragma unroll
    for (int q = 0; q < kNM; ++q) {
        const double v = wave_sum(acc[q]);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][q] = v;
    }
    __syncthreads();
    if (threadIdx.x < kNM)
        partial[(long long)blockIdx.x * kNM + threadIdx.x] =
            (red[0][threadIdx.x] + red[1][threadIdx.x]) + (red[2][threadIdx.x] + red[3][threadIdx.x]);
}

// Q_lm = h^3 sum of the workgroup partials (fixed order); zero beyond lmax
__global__ void __launch_bounds__(kPT) moments_finish(const double *__restrict__ partial, int nparts, double h3,
                                                      int lmax, double *__restrict__ Q)
{
    const int q = threadIdx.x;
    if (q >= kNM) return;
    double v = 0.0;
#pragma unroll 16
    for (int b = 0; b < nparts; ++b) v += partial[(long long)b * kNM + q];
    const int l = (int)sqrtf((float)q + 0.5f);
    Q[q] = l <= lmax ? h3 * v : 0.0;
}

struct SlabGeo {
    int no;
    long long off[6];  // start of face f = 2 ax + side in the slab array
    int nu[3], nv[3];  // extent of the face coordinates (u, v) for axis ax
};

// phi of Eq. phi:BC:discrete at the off-grid nodes: face f = 2 ax + side,
// layer L = 1..no (index ax = -L on the low side, n_ax - 1 + L on the high
// side), the other two indices over the grid in order
__global__ void __launch_bounds__(kPT) slab_kernel(const GridGeo g, const SlabGeo sg, const HarmNorm nrm, int lmax,
                                                   const double *__restrict__ Q, double *__restrict__ slab,
                                                   long long total)
{
    const long long t = blockIdx.x * (long long)kPT + threadIdx.x;
    if (t >= total) return;
    int f = 0;
    while (f < 5 && t >= sg.off[f + 1]) ++f;
    const int ax = f >> 1, side = f & 1;
    const long long loc = t - sg.off[f];
    const long long per = (long long)sg.nu[ax] * sg.nv[ax];
    const int L = (int)(loc / per) + 1;
    const long long uv = loc % per;
    const int u = (int)(uv / sg.nv[ax]), v = (int)(uv % sg.nv[ax]);
    const int nax = ax == 0 ? g.n0 : (ax == 1 ? g.n1 : g.n2);
    const int ia = side ? nax - 1 + L : -L;
    int idx[3];
    idx[ax] = ia;
    idx[ax == 0 ? 1 : 0] = u;
    idx[ax == 2 ? 1 : 2] = v;
    const double x = (idx[0] + 1) * g.h - g.c0, y = (idx[1] + 1) * g.h - g.c1, z = (idx[2] + 1) * g.h - g.c2;
    double R[kNM];
    solid_harmonics(x, y, z, nrm, R);
    const double r2 = x * x + y * y + z * z;
    const double rinv2 = 1.0 / r2;
    double rl = 1.0 / sqrt(r2);  // 1 / r^(2l+1), starting at l = 0
    double phi = 0.0;
    // Q is zero beyond lmax, so the fixed-length loops add exact zeros there
#pragma unroll
    for (int l = 0; l <= kLmax; ++l) {
        double s = 0.0;
#pragma unroll
        for (int m = -l; m <= l; ++m) s += Q[l * l + l + m] * R[l * l + l + m];
        phi += kFourPi / (2 * l + 1) * rl * s;
        rl *= rinv2;
    }
    (void)lmax;
    slab[t] = phi;
}

// rhs = c - d, d = -(1/4 pi) sum of w_p phi at the off-grid neighbours
// (Eq. Phi:correction); partial sums of rhs^2 per workgroup
__global__ void __launch_bounds__(kPT) rhs_kernel(const double *__restrict__ charge, const GridGeo g,
                                                  const SlabGeo sg, const double *__restrict__ w,
                                                  const double *__restrict__ slab, double *__restrict__ rhs,
                                                  double *__restrict__ part_bb)
{
    __shared__ double red[4];
    double bb = 0.0;
    for (long long t = blockIdx.x * (long long)kPT + threadIdx.x; t < g.nd; t += (long long)gridDim.x * kPT) {
        int id[3];
        double x, y, z;
        node_pos(g, t, id[0], id[1], id[2], x, y, z);
        const int nn[3] = {g.n0, g.n1, g.n2};
        double d = 0.0;
        for (int ax = 0; ax < 3; ++ax) {
            const int ia = id[ax];
            if (ia >= sg.no && ia < nn[ax] - sg.no) continue;
            const int u = id[ax == 0 ? 1 : 0], v = id[ax == 2 ? 1 : 2];
            const long long per = (long long)sg.nu[ax] * sg.nv[ax];
            const long long uv = (long long)u * sg.nv[ax] + v;
            for (int p = 1; p <= sg.no; ++p) {
                if (ia - p < 0) d += w[p] * slab[sg.off[2 * ax] + (long long)(p - ia - 1) * per + uv];
                if (ia + p > nn[ax] - 1) d += w[p] * slab[sg.off[2 * ax + 1] + (long long)(ia + p - nn[ax]) * per + uv];
            }
        }
        const double rv = charge[t] + d / kFourPi;
        rhs[t] = rv;
        bb += rv * rv;
    }
    const double s = block_sum(bb, red);
    if (threadIdx.x == 0) part_bb[blockIdx.x] = s;
}

__global__ void __launch_bounds__(kPT) axpy_kernel(double *__restrict__ r, const double *__restrict__ q, double a,
                                                   long long n)
{
    for (long long t = blockIdx.x * (long long)kPT + threadIdx.x; t < n; t += (long long)gridDim.x * kPT) r[t] += a * q[t];
}

__global__ void __launch_bounds__(kPT) fill_kernel(double *__restrict__ x, long long n)
{
    for (long long t = blockIdx.x * (long long)kPT + threadIdx.x; t < n; t += (long long)gridDim.x * kPT) x[t] = 0.0;
}

struct BjGeo {
    int n0, n1, n2;
    int b[3];     // block edge per axis
    int nb[3];    // blocks per axis
    int last[3];  // edge of the last block per axis
    int maxm;     // b0 b1 b2
    long long nblocks;
};

// the shape code of block (bi, bj, bk): bit 2/1/0 set when it is the last
// block of a ragged axis
__device__ __forceinline__ int bj_shape(const BjGeo &q, int bi, int bj, int bk, int (&dim)[3])
{
    const int bidx[3] = {bi, bj, bk};
    int code = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const bool lastb = bidx[a] == q.nb[a] - 1;
        dim[a] = lastb ? q.last[a] : q.b[a];
        code = 2 * code + (lastb ? 1 : 0);
    }
    return code;
}

// block-Jacobi step over all blocks.  A workgroup takes a brick of G = 256 /
// (b0 b1 b2) blocks that follow each other along z in one (block x, block y)
// row, so its global accesses are rows of G b2 consecutive nodes (coalesced):
// thread t owns node (a, b, zz) of the brick, t = (a b1 + b) G b2 + zz.  The
// residual goes through LDS into block order, thread (slot, row) forms row
// `row` of M^-1 r for block `slot` (sum over j ascending; the interior
// blocks' inverse read from LDS), and the result goes back through LDS to the
// brick order for the coalesced store.
// UPDATE: alpha = rz / pq, r -= alpha q; both modes: z = M^-1 r per block,
// p = z (INIT only), partials of r.z and r.r
template <bool UPDATE>
__global__ void __launch_bounds__(kPT)
    bj_kernel(const BjGeo q, const double *__restrict__ minv, double *__restrict__ r, double *__restrict__ p,
              const double *__restrict__ qv, double *__restrict__ z, const double *__restrict__ part_pq, int n_pq,
              double *__restrict__ part_rz, double *__restrict__ part_rr, int iter, PcgState *__restrict__ state)
{
    __shared__ double red[4];
    __shared__ double rs[kPT];
    __shared__ double zs[kPT];
    // the inverse of the interior block shape (code 0), read by every row of
    // every interior block, staged once per workgroup (blocks of at most
    // kBjStage nodes)
    __shared__ double sM[kBjStage * kBjStage];
    if (UPDATE && state->done < iter) return;
    const bool staged = q.maxm <= kBjStage;
    if (staged)
        for (int e = threadIdx.x; e < q.maxm * q.maxm; e += kPT) sM[e] = minv[e];
    double alpha = 0.0;
    if (UPDATE) {
        alpha = state->rz[iter & 1] / sum_partials(part_pq, n_pq, red);
        if (blockIdx.x == 0 && threadIdx.x == 0) state->alpha = alpha;
    }
    const int G = kPT / q.maxm;          // blocks per brick
    const int bpr = (q.nb[2] + G - 1) / G;  // bricks per (block x, block y) row
    const long long nbricks = (long long)q.nb[0] * q.nb[1] * bpr;
    // brick-order coordinates of this thread
    const int zw = G * q.b[2];
    const int ta = threadIdx.x / (q.b[1] * zw), tb = (threadIdx.x / zw) % q.b[1], tz = threadIdx.x % zw;
    const bool tin = threadIdx.x < q.b[0] * q.b[1] * zw;
    const int tslot = tz / q.b[2], tzl = tz % q.b[2];
    // block-order coordinates of this thread (compute phase)
    const int cslot = threadIdx.x / q.maxm, crow = threadIdx.x % q.maxm;
    double arz = 0.0, arr = 0.0;
    for (long long br = blockIdx.x; br < nbricks; br += gridDim.x) {
        const int bk0 = (int)(br % bpr) * G;
        const long long u = br / bpr;
        const int bj = (int)(u % q.nb[1]), bi = (int)(u / q.nb[1]);
        // load phase: this thread's node of the brick
        int dim[3] = {1, 1, 1};
        bool act = tin && bk0 + tslot < q.nb[2];
        long long node = 0;
        int lrow = 0;
        if (act) {
            (void)bj_shape(q, bi, bj, bk0 + tslot, dim);
            act = ta < dim[0] && tb < dim[1] && tzl < dim[2];
            lrow = (ta * dim[1] + tb) * dim[2] + tzl;
            node = ((long long)(bi * q.b[0] + ta) * q.n1 + (bj * q.b[1] + tb)) * q.n2 + ((bk0 + tslot) * q.b[2] + tzl);
        }
        double rv = 0.0;
        if (act) {
            if (UPDATE) {
                rv = r[node] - alpha * qv[node];
                r[node] = rv;
            } else {
                rv = r[node];
            }
            rs[tslot * q.maxm + lrow] = rv;
        }
        __syncthreads();
        // compute phase: row crow of block cslot
        if (cslot < G && bk0 + cslot < q.nb[2]) {
            int cd[3];
            const int code = bj_shape(q, bi, bj, bk0 + cslot, cd);
            const int m = cd[0] * cd[1] * cd[2];
            if (crow < m) {
                const double *rb = rs + cslot * q.maxm;
                double zv = 0.0;
                if (staged && code == 0) {
#pragma unroll 8
                    for (int j = 0; j < m; ++j) zv += sM[j * m + crow] * rb[j];
                } else {
                    const double *M = minv + (long long)code * q.maxm * q.maxm;
#pragma unroll 8
                    for (int j = 0; j < m; ++j) zv += M[(long long)j * m + crow] * rb[j];
                }
                zs[cslot * q.maxm + crow] = zv;
            }
        }
        __syncthreads();
        // store phase, brick order again
        if (act) {
            const double zv = zs[tslot * q.maxm + lrow];
            z[node] = zv;
            if (!UPDATE) p[node] = zv;
            arz += rv * zv;
            arr += rv * rv;
        }
        __syncthreads();
    }
    const double s1 = block_sum(arz, red);
    const double s2 = block_sum(arr, red);
    if (threadIdx.x == 0) {
        part_rz[blockIdx.x] = s1;
        part_rr[blockIdx.x] = s2;
    }
}

// Block-Jacobi step for blocks of 4 x 4 x 4 nodes in the eigenbasis of the
// block.  A restricted to a box of nodes is the sum of one small matrix per
// axis, T_x + T_y + T_z (Kronecker sum), T_m the m x m corner of the banded 1D
// operator; with T_m = U_m diag(l) U_m^T its inverse is three 4 x 4 products
// along the axes, a division by l_x + l_y + l_z and the three transposed
// products: 24 multiply-adds per node instead of the 64 of the dense inverse.
// Blocks cut short use the U_m of their extents, padded with zeros.
//
// Four lanes own a block, lane a its plane x = a (16 nodes); the x products
// exchange values within the quad of lanes (DPP), nothing goes through LDS but
// the tables.  Consecutive quads take blocks that follow each other along z,
// so a wave reads and writes rows of 512 bytes.
// What bounds it: r, q in, r, z out, 32 bytes per node (4.5 TB/s at 160^3).  Per
// application, 160^3: 29 us; dense inverses from LDS 75 us (with the x update,
// now in xp_update_kernel), dense inverses on the matrix cores 40 us; 96^3 11
// and 19 us.  Two waves per SIMD hold the 208 registers; at three or four the
// products spill (94 and 97 instead of 80 us per CG iteration).
constexpr int kDiagTab = 5 * 20;  // per m = 0..4: U_m (16 values, row i, column of the eigenvector j at 4 i + j), l (4)

// the value of quad lane J in every lane of the quad
template <int J>
__device__ __forceinline__ double quad_bcast(double v)
{
    constexpr int ctrl = J | (J << 2) | (J << 4) | (J << 6);
    union {
        double d;
        int i[2];
    } u;
    u.d = v;
    u.i[0] = __builtin_amdgcn_mov_dpp(u.i[0], ctrl, 0xf, 0xf, true);
    u.i[1] = __builtin_amdgcn_mov_dpp(u.i[1], ctrl, 0xf, 0xf, true);
    return u.d;
}

// v <- sum_j c[j] (v of quad lane j)
__device__ __forceinline__ void quad_product(double (&v)[4][4], const double (&c)[4])
{
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double x = v[i][k];
            v[i][k] = c[0] * quad_bcast<0>(x) + c[1] * quad_bcast<1>(x) + c[2] * quad_bcast<2>(x) +
                      c[3] * quad_bcast<3>(x);
        }
}

// along z (ROW) or y of the lane's plane: v <- U^T v (FWD) or U v
template <bool ROW, bool FWD>
__device__ __forceinline__ void axis_product(double (&v)[4][4], const double *U)
{
    // keep the tables in LDS between products (registers decide the waves in flight)
    asm volatile("" ::: "memory");
    double u[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) u[e] = U[e];
#pragma unroll
    for (int o = 0; o < 4; ++o) {
        double x[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) x[i] = ROW ? v[o][i] : v[i][o];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            double t = 0.0;
#pragma unroll
            for (int i = 0; i < 4; ++i) t += (FWD ? u[4 * i + j] : u[4 * j + i]) * x[i];
            if (ROW)
                v[o][j] = t;
            else
                v[j][o] = t;
        }
    }
}

// dinv: 1 / (l_x + l_y + l_z) per extents (m_x, m_y, m_z) = 1..4 each, [64][a][b][c]
template <bool UPDATE>
__global__ void __launch_bounds__(kPT, 2)
    bj_diag_kernel(const BjGeo q, const double *__restrict__ tab, const double *__restrict__ dinv,
                   double *__restrict__ r, double *__restrict__ p, const double *__restrict__ qv,
                   double *__restrict__ z, const double *__restrict__ part_pq, int n_pq, double *__restrict__ part_rz,
                   double *__restrict__ part_rr, int iter, PcgState *__restrict__ state)
{
    typedef double V4 __attribute__((ext_vector_type(4), aligned(8)));
    __shared__ double red[4];
    __shared__ double sU[kDiagTab];
    if (UPDATE && state->done < iter) return;
    if (threadIdx.x < kDiagTab) sU[threadIdx.x] = tab[threadIdx.x];
    double alpha = 0.0;
    if (UPDATE) {
        alpha = state->rz[iter & 1] / sum_partials(part_pq, n_pq, red);
        if (blockIdx.x == 0 && threadIdx.x == 0) state->alpha = alpha;
    } else {
        __syncthreads();
    }
    const int a = threadIdx.x & 3;
    double arz = 0.0, arr = 0.0;
    for (long long blk = (blockIdx.x * (long long)kPT + threadIdx.x) >> 2; blk < q.nblocks;
         blk += (long long)gridDim.x * (kPT / 4)) {
        const int bk = (int)(blk % q.nb[2]);
        const long long u = blk / q.nb[2];
        const int bj = (int)(u % q.nb[1]), bi = (int)(u / q.nb[1]);
        const int mx = bi == q.nb[0] - 1 ? q.last[0] : 4;
        const int my = bj == q.nb[1] - 1 ? q.last[1] : 4;
        const int mz = bk == q.nb[2] - 1 ? q.last[2] : 4;
        const long long n0 = ((long long)(4 * bi + a) * q.n1 + 4 * bj) * q.n2 + 4 * bk;
        const bool whole = a < mx && mz == 4;
        double v[4][4];
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int c = 0; c < 4; ++c) v[b][c] = 0.0;
        if (whole) {
#pragma unroll
            for (int b = 0; b < 4; ++b)
                if (b < my) {
                    const long long n = n0 + (long long)b * q.n2;
                    V4 x = *(const V4 *)(r + n);
                    if (UPDATE) {
                        const V4 y = *(const V4 *)(qv + n);
#pragma unroll
                        for (int c = 0; c < 4; ++c) x[c] -= alpha * y[c];
                        *(V4 *)(r + n) = x;
                    }
#pragma unroll
                    for (int c = 0; c < 4; ++c) v[b][c] = x[c];
                }
        } else if (a < mx) {
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    if (b < my && c < mz) {
                        const long long n = n0 + (long long)b * q.n2 + c;
                        double x = r[n];
                        if (UPDATE) {
                            x -= alpha * qv[n];
                            r[n] = x;
                        }
                        v[b][c] = x;
                    }
        }
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int c = 0; c < 4; ++c) arr += v[b][c] * v[b][c];
        const double *Ux = sU + 20 * mx, *Uy = sU + 20 * my, *Uz = sU + 20 * mz;
        axis_product<true, true>(v, Uz);
        axis_product<false, true>(v, Uy);
        {
            const double c[4] = {Ux[a], Ux[4 + a], Ux[8 + a], Ux[12 + a]};
            quad_product(v, c);
        }
        asm volatile("" ::: "memory");
        const double *d = dinv + (((mx - 1) * 4 + (my - 1)) * 4 + (mz - 1)) * 64 + 16 * a;
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const double t = v[b][c] * d[4 * b + c];
                arz += v[b][c] * t;  // r.z = sum of squares over the eigenvalues
                v[b][c] = t;
            }
        {
            const double c[4] = {Ux[4 * a], Ux[4 * a + 1], Ux[4 * a + 2], Ux[4 * a + 3]};
            quad_product(v, c);
        }
        axis_product<false, false>(v, Uy);
        axis_product<true, false>(v, Uz);
        if (whole) {
#pragma unroll
            for (int b = 0; b < 4; ++b)
                if (b < my) {
                    const long long n = n0 + (long long)b * q.n2;
                    const V4 x = {v[b][0], v[b][1], v[b][2], v[b][3]};
                    *(V4 *)(z + n) = x;
                    if (!UPDATE) *(V4 *)(p + n) = x;
                }
        } else if (a < mx) {
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    if (b < my && c < mz) {
                        const long long n = n0 + (long long)b * q.n2 + c;
                        z[n] = v[b][c];
                        if (!UPDATE) p[n] = v[b][c];
                    }
        }
    }
    const double s1 = block_sum(arz, red);
    const double s2 = block_sum(arr, red);
    if (threadIdx.x == 0) {
        part_rz[blockIdx.x] = s1;
        part_rr[blockIdx.x] = s2;
    }
}

// partials of p.q
__global__ void __launch_bounds__(kPT) dot_kernel(const double *__restrict__ a, const double *__restrict__ b,
                                                  long long n, double *__restrict__ part, int iter,
                                                  const PcgState *__restrict__ state)
{
    __shared__ double red[4];
    if (state->done < iter) return;
    double s = 0.0;
    for (long long t = blockIdx.x * (long long)kPT + threadIdx.x; t < n; t += (long long)gridDim.x * kPT) s += a[t] * b[t];
    s = block_sum(s, red);
    if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// x += alpha p, the convergence test and p = z + beta p, beta = rz_new / rz
__global__ void __launch_bounds__(kPT)
    xp_update_kernel(double *__restrict__ x, double *__restrict__ p, const double *__restrict__ z, long long n,
                     const double *__restrict__ rz_new, const double *__restrict__ rr, int nbj, double tol2, int iter,
                     PcgState *__restrict__ state)
{
    __shared__ double red[8];
    if (state->done < iter) return;
    const double alpha = state->alpha, rz_old = state->rz[iter & 1], bb = state->bb;
    double rrv, rzv;
    sum_partials2(rr, rz_new, nbj, red, rrv, rzv);
    const bool done = rrv <= tol2 * bb;
    const double beta = rzv / rz_old;
    const long long step = (long long)gridDim.x * kPT, t0 = blockIdx.x * (long long)kPT + threadIdx.x;
    // pairs of nodes, 16 bytes per access
    typedef double v2d __attribute__((ext_vector_type(2), aligned(8)));
    const long long n2 = n / 2;
    for (long long t = t0; t < n2; t += step) {
        const v2d pv = ((const v2d *)p)[t];
        v2d xv = ((const v2d *)x)[t];
        xv[0] += alpha * pv[0];
        xv[1] += alpha * pv[1];
        ((v2d *)x)[t] = xv;
        if (!done) {
            v2d zv = ((const v2d *)z)[t];
            zv[0] += beta * pv[0];
            zv[1] += beta * pv[1];
            ((v2d *)p)[t] = zv;
        }
    }
    if ((n & 1) && t0 == 0) {
        const double pv = p[n - 1];
        x[n - 1] += alpha * pv;
        if (!done) p[n - 1] = z[n - 1] + beta * pv;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (done) state->done = iter;
        state->iters = iter + 1;
        state->rr = rrv;
        state->rz[1 - (iter & 1)] = rzv;
    }
}

// state after the initial residual: converged already when r.r <= tol^2 b.b
__global__ void __launch_bounds__(kPT) pcg_start_kernel(const double *__restrict__ rr, const double *__restrict__ rz,
                                                        int nbj, const double *__restrict__ part_bb, int nbb,
                                                        double tol2, PcgState *__restrict__ state)
{
    __shared__ double red[4];
    const double rrv = sum_partials(rr, nbj, red);
    const double rzv = sum_partials(rz, nbj, red);
    const double bb = sum_partials(part_bb, nbb, red);
    if (threadIdx.x == 0) {
        state->done = rrv <= tol2 * bb ? -1 : kNotDone;
        state->iters = 0;
        state->rr = rrv;
        state->bb = bb;
        state->rz[0] = rzv;
    }
}

// Gauss-Jordan inverse of an SPD matrix (host, FP64, partial pivoting)
bool invert(std::vector<double> &A, int m)
{
    std::vector<double> I((size_t)m * m, 0.0);
    for (int i = 0; i < m; ++i) I[(size_t)i * m + i] = 1.0;
    for (int c = 0; c < m; ++c) {
        int piv = c;
        for (int r = c + 1; r < m; ++r)
            if (std::fabs(A[(size_t)r * m + c]) > std::fabs(A[(size_t)piv * m + c])) piv = r;
        if (A[(size_t)piv * m + c] == 0.0) return false;
        if (piv != c)
            for (int k = 0; k < m; ++k) {
                std::swap(A[(size_t)c * m + k], A[(size_t)piv * m + k]);
                std::swap(I[(size_t)c * m + k], I[(size_t)piv * m + k]);
            }
        const double d = A[(size_t)c * m + c];
        for (int k = 0; k < m; ++k) {
            A[(size_t)c * m + k] /= d;
            I[(size_t)c * m + k] /= d;
        }
        for (int r = 0; r < m; ++r) {
            if (r == c) continue;
            const double f = A[(size_t)r * m + c];
            if (f == 0.0) continue;
            for (int k = 0; k < m; ++k) {
                A[(size_t)r * m + k] -= f * A[(size_t)c * m + k];
                I[(size_t)r * m + k] -= f * I[(size_t)c * m + k];
            }
        }
    }
    A.swap(I);
    return true;
}

// eigenvalues l and eigenvectors (columns of U, m x m row-major in a 4 x 4
// array) of a symmetric m x m matrix, m <= 4: cyclic Jacobi rotations
void small_eigen(double (&A)[4][4], int m, double (&U)[4][4], double (&l)[4])
{
    for (int i = 0; i < 4; ++i)
        for (int j = 0; j < 4; ++j) U[i][j] = i == j && i < m ? 1.0 : 0.0;
    for (int sweep = 0; sweep < 30; ++sweep) {
        double off = 0.0;
        for (int p = 0; p < m; ++p)
            for (int q = p + 1; q < m; ++q) off += A[p][q] * A[p][q];
        if (off == 0.0) break;
        for (int p = 0; p < m; ++p)
            for (int q = p + 1; q < m; ++q) {
                if (A[p][q] == 0.0) continue;
                const double tau = (A[q][q] - A[p][p]) / (2.0 * A[p][q]);
                const double t = (tau >= 0 ? 1.0 : -1.0) / (std::fabs(tau) + std::sqrt(1.0 + tau * tau));
                const double c = 1.0 / std::sqrt(1.0 + t * t), s = t * c;
                for (int k = 0; k < m; ++k) {  // columns p, q of A and U
                    const double x = A[k][p], y = A[k][q];
                    A[k][p] = c * x - s * y;
                    A[k][q] = s * x + c * y;
                    const double a = U[k][p], b = U[k][q];
                    U[k][p] = c * a - s * b;
                    U[k][q] = s * a + c * b;
                }
                for (int k = 0; k < m; ++k) {  // rows
                    const double x = A[p][k], y = A[q][k];
                    A[p][k] = c * x - s * y;
                    A[q][k] = s * x + c * y;
                }
                A[p][q] = A[q][p] = 0.0;
            }
    }
    for (int i = 0; i < 4; ++i) l[i] = i < m ? A[i][i] : 1.0;
}

size_t al(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace
}  // namespace sparc

using namespace sparc;

struct sparc_poisson {
    int device = 0;
    GridGeo g{};
    SlabGeo sg{};
    BjGeo bj{};
    int lmax = 6;
    int radius = 6;
    sparc_op *op0 = nullptr;  // zero potential, no atoms: its step kernel applies -1/2 lap_h
    HarmNorm nrm{};
    double *d_minv = nullptr;
    bool diag = false;  // blocks of 4 x 4 x 4 nodes: d_minv holds the tables of bj_diag_kernel
    double *d_w = nullptr;
    long long slab_total = 0;
    int nmom = 0, nred = 0, nbjg = 0, npq = 0;  // workgroups of the moment, reduction and block-Jacobi kernels
};

namespace {

struct PoisWs {
    double *r, *z, *p, *q, *slab, *mpart, *Q, *bb, *pq, *rz, *rr;
    PcgState *state;
    size_t total;
};

PoisWs carve(const sparc_poisson *P, void *ws)
{
    PoisWs W{};
    char *b = (char *)ws;
    size_t o = 0;
    auto take = [&](size_t bytes) {
        char *p = b ? b + o : nullptr;
        o += al(bytes);
        return p;
    };
    const size_t vec = (size_t)P->g.nd * sizeof(double);
    W.r = (double *)take(vec);
    W.z = (double *)take(vec);
    W.p = (double *)take(vec);
    W.q = (double *)take(vec);
    W.slab = (double *)take((size_t)P->slab_total * sizeof(double));
    W.mpart = (double *)take((size_t)P->nmom * kNM * sizeof(double));
    W.Q = (double *)take(kNM * sizeof(double));
    W.bb = (double *)take(kRedMax * sizeof(double));
    W.pq = (double *)take((size_t)std::max(P->npq, kRedMax) * sizeof(double));
    W.rz = (double *)take(kRedMax * sizeof(double));
    W.rr = (double *)take(kRedMax * sizeof(double));
    W.state = (PcgState *)take(sizeof(PcgState));
    W.total = o;
    return W;
}

}  // namespace

extern "C" int sparc_poisson_create(const sparc_grid *grid, int32_t lmax, const int32_t *block, sparc_poisson **out)
{
    if (!grid || !out) return fail(SPARC_E_ARG, "null argument");
    *out = nullptr;
    if (lmax < 0 || lmax > kLmax) return fail(SPARC_E_ARG, "lmax must be in 0..6");
    int b[3] = {4, 4, 4};
    if (block)
        for (int a = 0; a < 3; ++a) b[a] = block[a];
    for (int a = 0; a < 3; ++a)
        if (b[a] < 1 || b[a] > 8) return fail(SPARC_E_ARG, "block edges must be in 1..8");
    if (b[0] * b[1] * b[2] > kPT) return fail(SPARC_E_ARG, "a block may hold at most 256 nodes");
    const int64_t nd = (int64_t)grid->n[0] * grid->n[1] * grid->n[2];
    std::vector<double> zero(nd > 0 ? nd : 1, 0.0);
    sparc_op *op0 = nullptr;
    int st = sparc_op_create(grid, zero.data(), 0, nullptr, &op0);  // validates the grid
    if (st) return st;
    sparc_poisson *P = new (std::nothrow) sparc_poisson();
    if (!P) {
        sparc_op_destroy(op0);
        return fail(SPARC_E_NOMEM, "host allocation failed");
    }
    P->op0 = op0;
    (void)hipGetDevice(&P->device);
    P->lmax = lmax;
    P->radius = grid->radius;
    const int n[3] = {grid->n[0], grid->n[1], grid->n[2]};
    P->g = {n[0], n[1], n[2], (long long)nd, grid->h, 0.5 * (n[0] + 1) * grid->h, 0.5 * (n[1] + 1) * grid->h,
            0.5 * (n[2] + 1) * grid->h};
    // solid-harmonic normalisation: sqrt((2l+1)/(4 pi) (l-m)!/(l+m)!), times sqrt 2 for m != 0
    for (int l = 0; l <= kLmax; ++l)
        for (int m = 0; m <= l; ++m) {
            double ratio = 1.0;
            for (int k = l - m + 1; k <= l + m; ++k) ratio /= k;
            double c = std::sqrt((2 * l + 1) / kFourPi * ratio);
            if (m > 0) c *= std::sqrt(2.0);
            P->nrm.c[l * l + l + m] = c;
            P->nrm.c[l * l + l - m] = c;
        }
    // off-grid slabs
    SlabGeo &sg = P->sg;
    sg.no = grid->radius;
    long long off = 0;
    for (int ax = 0; ax < 3; ++ax) {
        sg.nu[ax] = n[ax == 0 ? 1 : 0];
        sg.nv[ax] = n[ax == 2 ? 1 : 2];
        for (int side = 0; side < 2; ++side) {
            sg.off[2 * ax + side] = off;
            off += (long long)sg.no * sg.nu[ax] * sg.nv[ax];
        }
    }
    P->slab_total = off;
    // block Jacobi: dense inverse of A restricted to each block shape
    BjGeo &q = P->bj;
    q.n0 = n[0];
    q.n1 = n[1];
    q.n2 = n[2];
    q.nblocks = 1;
    for (int a = 0; a < 3; ++a) {
        q.b[a] = std::min(b[a], n[a]);
        q.nb[a] = (n[a] + q.b[a] - 1) / q.b[a];
        q.last[a] = n[a] - (q.nb[a] - 1) * q.b[a];
        q.nblocks *= q.nb[a];
    }
    q.maxm = q.b[0] * q.b[1] * q.b[2];
    const double *w = op0->w;
    P->diag = b[0] == 4 && b[1] == 4 && b[2] == 4;
    std::vector<double> minv;
    if (P->diag) {
        minv.assign(kDiagTab + 64 * 64, 0.0);
        for (int m = 1; m <= 4; ++m) {
            double T[4][4] = {}, U[4][4], l[4];
            for (int i = 0; i < m; ++i)
                for (int j = 0; j < m; ++j) {
                    const int p = std::abs(i - j);
                    T[i][j] = p > grid->radius ? 0.0 : (p == 0 ? 2.0 : 1.0) * w[p] * (-1.0 / kFourPi);
                }
            small_eigen(T, m, U, l);
            for (int i = 0; i < 4; ++i) {
                for (int j = 0; j < 4; ++j) minv[20 * m + 4 * i + j] = U[i][j];
                minv[20 * m + 16 + i] = l[i];
            }
        }
        for (int e = 0; e < 64 * 64; ++e) {
            const int m[3] = {e / 1024 + 1, e / 256 % 4 + 1, e / 64 % 4 + 1}, i[3] = {e / 16 % 4, e / 4 % 4, e % 4};
            double sum = 0.0;
            for (int d = 0; d < 3; ++d) sum += minv[20 * m[d] + 16 + i[d]];
            minv[kDiagTab + e] = 1.0 / sum;
        }
    } else {
        minv.assign((size_t)8 * q.maxm * q.maxm, 0.0);
        for (int code = 0; code < 8; ++code) {
            int dim[3];
            for (int a = 0; a < 3; ++a) dim[a] = (code >> (2 - a)) & 1 ? q.last[a] : q.b[a];
            const int m = dim[0] * dim[1] * dim[2];
            std::vector<double> A((size_t)m * m, 0.0);
            for (int t = 0; t < m; ++t) {
                const int c[3] = {t / (dim[1] * dim[2]), (t / dim[2]) % dim[1], t % dim[2]};
                A[(size_t)t * m + t] += 6.0 * w[0];
                for (int a = 0; a < 3; ++a)
                    for (int p = 1; p <= grid->radius; ++p)
                        for (int s = -1; s <= 1; s += 2) {
                            int e[3] = {c[0], c[1], c[2]};
                            e[a] += s * p;
                            if (e[a] < 0 || e[a] >= dim[a]) continue;
                            A[(size_t)t * m + (e[0] * dim[1] + e[1]) * dim[2] + e[2]] += w[p];
                        }
            }
            for (double &v : A) v *= -1.0 / kFourPi;
            if (!invert(A, m)) {
                sparc_poisson_destroy(P);
                return fail(SPARC_E_HIP, "block matrix is singular");
            }
            // symmetrise (the inverse of a symmetric matrix; removes rounding asymmetry)
            for (int i = 0; i < m; ++i)
                for (int j = i + 1; j < m; ++j) {
                    const double s = 0.5 * (A[(size_t)i * m + j] + A[(size_t)j * m + i]);
                    A[(size_t)i * m + j] = A[(size_t)j * m + i] = s;
                }
            std::copy(A.begin(), A.end(), minv.begin() + (size_t)code * q.maxm * q.maxm);
        }
    }
    std::vector<double> wv(kMaxRadius + 1, 0.0);
    for (int p = 0; p <= grid->radius; ++p) wv[p] = w[p];
    if (hipMalloc(&P->d_minv, minv.size() * sizeof(double)) != hipSuccess ||
        hipMalloc(&P->d_w, wv.size() * sizeof(double)) != hipSuccess) {
        sparc_poisson_destroy(P);
        return fail(SPARC_E_NOMEM, "device allocation failed");
    }
    if (hipMemcpy(P->d_minv, minv.data(), minv.size() * sizeof(double), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(P->d_w, wv.data(), wv.size() * sizeof(double), hipMemcpyHostToDevice) != hipSuccess) {
        sparc_poisson_destroy(P);
        return fail(SPARC_E_HIP, "copy of the block inverses failed");
    }
    // see sparc_op_create: a solve may run on a stream that does not wait for the null stream
    if (hipStreamSynchronize(0) != hipSuccess) {
        sparc_poisson_destroy(P);
        return fail(SPARC_E_HIP, "copies of the solver's data failed");
    }
    P->nmom = (int)std::max<long long>(1, std::min<long long>(256, (nd + kPT - 1) / kPT));
    P->nred = (int)std::max<long long>(1, std::min<long long>(kRedMax, (nd + 4 * kPT - 1) / (4 * kPT)));
    if (P->diag) {
        P->nbjg = (int)std::max<long long>(1, std::min<long long>(kRedMax, (4 * q.nblocks + kPT - 1) / kPT));
    } else {
        const int G = kPT / q.maxm;
        const long long bricks = (long long)q.nb[0] * q.nb[1] * ((q.nb[2] + G - 1) / G);
        P->nbjg = (int)std::max<long long>(1, std::min<long long>(kRedMax, bricks));
    }
    P->npq = vstep_takes(op0) ? (int)vstep_blocks(op0) : 0;
    *out = P;
    return SPARC_OK;
}

extern "C" int sparc_poisson_destroy(sparc_poisson *P)
{
    if (!P) return SPARC_OK;
    (void)hipFree(P->d_minv);
    (void)hipFree(P->d_w);
    sparc_op_destroy(P->op0);
    delete P;
    return SPARC_OK;
}

extern "C" size_t sparc_poisson_workspace_bytes(const sparc_poisson *P)
{
    if (!P) return 0;
    return carve(P, nullptr).total;
}

extern "C" int sparc_poisson_solve(sparc_poisson *P, const double *charge, double *phi, int32_t use_guess, double tol,
                                   int32_t max_iter, int32_t *iters, double *rel_resid, double *moments, void *ws,
                                   size_t ws_bytes, void *stream)
{
    if (!P || !charge || !phi) return fail(SPARC_E_ARG, "null argument");
    if (!(tol > 0.0) || max_iter < 0) return fail(SPARC_E_ARG, "need tol > 0 and max_iter >= 0");
    const PoisWs W = carve(P, ws);
    if (!ws || ws_bytes < W.total) return fail(SPARC_E_WORKSPACE, "workspace missing or too small");
    const long long nd = P->g.nd;
    const char *c0 = (const char *)charge, *c1 = c0 + nd * 8, *f0 = (const char *)phi, *f1 = f0 + nd * 8;
    const char *w0 = (const char *)ws, *w1 = w0 + W.total;
    if ((c0 < f1 && f0 < c1) || (w0 < f1 && f0 < w1) || (w0 < c1 && c0 < w1))
        return fail(SPARC_E_ALIAS, "charge, phi and the workspace must not overlap");
    TraceRange trace("sparc_poisson_solve");
    hipStream_t s = (hipStream_t)stream;
    const int nvec = P->nred;
    ProfScope prof(6, s);
    // multipole moments and the boundary values of phi
    hipLaunchKernelGGL(moments_kernel, dim3(P->nmom), dim3(kPT), 0, s, charge, P->g, P->nrm, W.mpart);
    hipLaunchKernelGGL(moments_finish, dim3(1), dim3(kPT), 0, s, (const double *)W.mpart, P->nmom,
                       P->g.h * P->g.h * P->g.h, P->lmax, W.Q);
    const long long sb = (P->slab_total + kPT - 1) / kPT;
    if (sb > 0x7fffffffLL) return fail(SPARC_E_SHAPE, "grid too large");
    hipLaunchKernelGGL(slab_kernel, dim3((unsigned)sb), dim3(kPT), 0, s, P->g, P->sg, P->nrm, P->lmax,
                       (const double *)W.Q, W.slab, P->slab_total);
    // right-hand side into r
    hipLaunchKernelGGL(rhs_kernel, dim3(nvec), dim3(kPT), 0, s, charge, P->g, P->sg, (const double *)P->d_w,
                       (const double *)W.slab, W.r, W.bb);
    const FLaunch V = choose_vec_launch(P->op0, SPARC_F64, 1, {nd, nd});
    const StepLaunch L = choose_step_launch(P->op0, SPARC_F64, 1);
    const StepCoef cA{1.0 / (2.0 * M_PI), 0.0, 0.0, 0};  // A = (1/2 pi)(-1/2 lap_h)
    int st;
    if (use_guess) {
        if ((st = launch_h_step(P->op0, SPARC_F64, phi, nd, nullptr, 0, W.q, nd, 1, nullptr, cA, L, s, &V))) return st;
        hipLaunchKernelGGL(axpy_kernel, dim3(nvec), dim3(kPT), 0, s, W.r, (const double *)W.q, -1.0, nd);
    } else {
        hipLaunchKernelGGL(fill_kernel, dim3(nvec), dim3(kPT), 0, s, phi, nd);
    }
    // one block-Jacobi launch: INIT or the update of iteration `it`
    const int npq = P->npq > 0 ? P->npq : nvec;
    auto block_jacobi = [&](bool update, int it) {
        const dim3 g(P->nbjg), b(kPT);
#define SPARC_BJ(kernel, ...)                                                                                \
    hipLaunchKernelGGL(kernel, g, b, 0, s, P->bj, (const double *)P->d_minv, __VA_ARGS__ W.r, W.p,           \
                       (const double *)W.q, W.z, (const double *)W.pq, npq, W.rz, W.rr, it, W.state)
        if (P->diag && update)
            SPARC_BJ(bj_diag_kernel<true>, (const double *)P->d_minv + kDiagTab, );
        else if (P->diag)
            SPARC_BJ(bj_diag_kernel<false>, (const double *)P->d_minv + kDiagTab, );
        else if (update)
            SPARC_BJ(bj_kernel<true>, );
        else
            SPARC_BJ(bj_kernel<false>, );
#undef SPARC_BJ
    };
    block_jacobi(false, 0);
    const double tol2 = tol * tol;
    hipLaunchKernelGGL(pcg_start_kernel, dim3(1), dim3(kPT), 0, s, (const double *)W.rr, (const double *)W.rz, P->nbjg,
                       (const double *)W.bb, nvec, tol2, W.state);
    SPARC_HIP(hipGetLastError());
    PcgState hs{};
    SPARC_HIP(hipMemcpyAsync(&hs, W.state, sizeof(hs), hipMemcpyDeviceToHost, s));
    SPARC_HIP(hipStreamSynchronize(s));
    int it = 0;
    while (hs.done == kNotDone && it < max_iter) {
        const int chunk = std::min(chunk_from(it, use_guess != 0), max_iter - it);
        for (int c = 0; c < chunk; ++c, ++it) {
            if (P->npq > 0) {
                if ((st = launch_vstep(P->op0, W.p, W.q, cA.alpha, W.pq, &W.state->done, it, s))) return st;
            } else {
                if ((st = launch_h_step(P->op0, SPARC_F64, W.p, nd, nullptr, 0, W.q, nd, 1, nullptr, cA, L, s, &V)))
                    return st;
                hipLaunchKernelGGL(dot_kernel, dim3(nvec), dim3(kPT), 0, s, (const double *)W.p, (const double *)W.q, nd,
                                   W.pq, it, (const PcgState *)W.state);
            }
            block_jacobi(true, it);
            hipLaunchKernelGGL(xp_update_kernel, dim3(nvec), dim3(kPT), 0, s, phi, W.p, (const double *)W.z, nd,
                               (const double *)W.rz, (const double *)W.rr, P->nbjg, tol2, it, W.state);
        }
        SPARC_HIP(hipGetLastError());
        SPARC_HIP(hipMemcpyAsync(&hs, W.state, sizeof(hs), hipMemcpyDeviceToHost, s));
        SPARC_HIP(hipStreamSynchronize(s));
    }
    if (moments) {
        SPARC_HIP(hipMemcpyAsync(moments, W.Q, (size_t)(P->lmax + 1) * (P->lmax + 1) * sizeof(double),
                                 hipMemcpyDeviceToHost, s));
        SPARC_HIP(hipStreamSynchronize(s));
    }
    if (iters) *iters = hs.iters;
    if (rel_resid) *rel_resid = hs.bb > 0 ? std::sqrt(hs.rr / hs.bb) : 0.0;
    return SPARC_OK;
}
