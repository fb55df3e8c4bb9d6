// Nonlocal component of the atomic forces (Sec. 3.6, Eqs.
// NonlocForce:Discrete and NonLocForce:U:W; Alg. 4):
//   f_J = -4 sum_n g_n sum_lm gamma_Jl Y_Jnlm W_Jnlm,
//   Y_Jnlm = h^3 sum_x psi_n chi_Jlm,  W_Jnlm = h^3 sum_x (grad_h psi_n) chi_Jlm,
// with grad_h the finite-difference gradient of Eq. gradient:approximate and
// zero Dirichlet padding.
//
// Design.  The paper forms grad_h psi_n on each atom's cube and contracts it
// with chi.  With zero padding the gradient matrix is antisymmetric, so
//   W_Jnlm[d] = h^3 sum_x psi_n(x) F_Jlm,d(x),  F_Jlm,d = -grad_h,d chi_Jlm,
// exactly: F lives on the cube widened by the stencil radius along d, is a
// property of the operator, and is built once (host, FP64) on the first call.
// Y and the three W components are then four projector-like contractions of
// the same nodes.  An atom's nodes are read once: the cube's rows, widened along
// z, with all 4 nproj functions as columns of the matrix product, then the arms
// that widen the cube along x and y with the one function set that is not zero
// there.  Large launches give an atom and 32 orbitals to one workgroup, which
// reduces its contractions to the three force components of its orbitals on
// the spot; small ones split the nodes over workgroups.  Either way a second
// kernel adds in a fixed order, so the forces are reproducible bit for bit.
// FP32 blocks are widened as they are loaded; all sums are FP64.
//
// What bounds it: the lines of the short node rows, 843 per atom and orbital at
// 160^3.  Orbital blocks run fastest, so that an atom's functions stay in the
// cache (2.24 against 2.38 ms with atoms fastest); two blocks of 16 orbitals
// share the function loads (2.38 against 2.78 ms with one).  128 atoms, 9
// projectors, 600 FP32 orbitals: 5.34 -> 2.26 ms (8.3 GB of lines at 3.7 TB/s);
// with the four boxes as records of their own it read 1701 lines per atom and
// orbital.  16 atoms x 200 orbitals at 96^3: 146 -> 72 us.
#include <algorithm>
#include <vector>

#include "nonlocal_kernel.hpp"

namespace sparc {
namespace {

// w~_1..w~_no of Eq. gradient:approximate, the factorial ratio accumulated as
// a product of q factors (no - q + i) / (no + i)
void gradient_weights(int no, double h, double *w)
{
    for (int q = 1; q <= no; ++q) {
        double ratio = 1.0;
        for (int i = 1; i <= q; ++i) ratio *= double(no - q + i) / double(no + i);
        w[q] = ((q & 1) ? 1.0 : -1.0) * ratio / (h * q);
    }
}

// one box of units of an atom with nf functions on it ([function][unit][4])
struct ForceBox {
    int unit0, nunits;
    long long fun0;
    int nf;
};
// the atom's boxes: the cube's rows widened along z with the functions chi, F_x,
// F_y, F_z (nproj each), and the arms along x and y with F_x and F_y
struct ForceAtom {
    ForceBox box[3];
    int nproj, proj0;
};

int build_force_tables(const sparc_op *op)
{
    const int natoms = op->natoms;
    const int R = op->radius;
    double w[kMaxRadius + 1] = {0};
    gradient_weights(R, op->h, w);
    int64_t chi_total = 0;
    for (const AtomDev &a : op->atoms) chi_total += (int64_t)a.ext[0] * a.ext[1] * a.ext[2] * a.nproj;
    std::vector<double> chi(chi_total);
    SPARC_HIP(hipMemcpy(chi.data(), op->d_chi64, chi_total * sizeof(double), hipMemcpyDeviceToHost));

    // the boxes' parts (the widened rows; the arms below and above the cube),
    // their units and the position of each of their nodes in the box
    struct Part {
        int lo[3], ext[3];
        std::vector<int> at;
    };
    std::vector<ForceAtom> rec(natoms);
    std::vector<std::vector<Part>> parts(3 * natoms);
    std::vector<int> units;
    size_t nfun = 0;
    for (int J = 0; J < natoms; ++J) {
        const AtomDev &A = op->atoms[J];
        ForceAtom &F = rec[J];
        F.nproj = A.nproj;
        F.proj0 = A.proj0;
        for (int k = 0; k < 3; ++k) {
            ForceBox &B = F.box[k];
            B.unit0 = (int)(units.size() / 2);
            B.fun0 = (long long)nfun;
            B.nf = k == 0 ? 4 * A.nproj : A.nproj;
            B.nunits = 0;
            auto part = [&](int axis, int from, int to) {
                from = std::max(from, 0);
                to = std::min(to, op->n[axis]);
                if (from >= to) return;
                Part P;
                for (int e = 0; e < 3; ++e) {
                    P.lo[e] = e == axis ? from : A.lo[e];
                    P.ext[e] = e == axis ? to - from : A.ext[e];
                }
                const int first = 4 * B.nunits;
                B.nunits += append_units(op->n, op->nd, P.lo, P.ext, units, P.at);
                for (int &o : P.at) o += first;
                parts[3 * J + k].push_back(std::move(P));
            };
            if (k == 0) {
                part(2, A.lo[2] - R, A.lo[2] + A.ext[2] + R);
                const Part &P = parts[3 * J].back();
                for (size_t t = 0; t < P.at.size(); ++t) {
                    const int z = P.lo[2] + (int)(t % P.ext[2]) - A.lo[2];
                    if (z < 0 || z >= A.ext[2]) units[2 * (B.unit0 + P.at[t] / 4) + 1] |= 16 << P.at[t] % 4;
                }
            } else {
                const int d = k - 1;
                part(d, A.lo[d] - R, A.lo[d]);
                part(d, A.lo[d] + A.ext[d], A.lo[d] + A.ext[d] + R);
            }
            if (units.size() > 0x7fffffffULL) return fail(SPARC_E_SHAPE, "force tables too large");
            nfun += 4 * (size_t)B.nunits * B.nf;
        }
    }
    // lanes past their share read their box's first unit: one more for an empty
    // box at the end of the table
    units.insert(units.end(), 2, 0);
    std::vector<double> fun(nfun, 0.0);
    for (int J = 0; J < natoms; ++J) {
        const AtomDev &A = op->atoms[J];
        const int st[3] = {A.ext[1] * A.ext[2], A.ext[2], 1};
        for (int k = 0; k < 3; ++k) {
            const ForceBox &B = rec[J].box[k];
            for (int f = 0; f < B.nf; ++f) {
                // r = 0: chi; r = 1 + d: -grad_d chi = sum_q w_q (chi(y - q e_d) - chi(y + q e_d)), chi 0 off the cube
                const int r = k == 0 ? f / A.nproj : k, p = f % A.nproj, d = r - 1;
                const double *c = chi.data() + A.chi0 + (int64_t)p * st[0] * A.ext[0];
                double *out = fun.data() + B.fun0 + 4 * (size_t)B.nunits * f;
                for (const Part &P : parts[3 * J + k]) {
                    size_t t = 0;
                    for (int i = 0; i < P.ext[0]; ++i)
                        for (int j = 0; j < P.ext[1]; ++j)
                            for (int l = 0; l < P.ext[2]; ++l, ++t) {
                                const int y[3] = {P.lo[0] + i - A.lo[0], P.lo[1] + j - A.lo[1], P.lo[2] + l - A.lo[2]};
                                bool in = true;
                                for (int e = 0; e < 3; ++e)
                                    if (e != d && (y[e] < 0 || y[e] >= A.ext[e])) in = false;
                                if (!in) continue;
                                const double *cy = c + y[0] * st[0] + y[1] * st[1] + y[2];
                                if (r == 0) {
                                    out[P.at[t]] = *cy;
                                    continue;
                                }
                                double v = 0.0;
                                for (int q = 1; q <= R; ++q) {
                                    const int a = y[d] - q, b = y[d] + q;
                                    v += w[q] * ((a >= 0 && a < A.ext[d] ? cy[-q * st[d]] : 0.0) -
                                                 (b >= 0 && b < A.ext[d] ? cy[q * st[d]] : 0.0));
                                }
                                out[P.at[t]] = v;
                            }
                }
            }
        }
    }
    std::vector<double> gam(op->gamma.begin(), op->gamma.end());
    if (hipMalloc(&op->d_fatoms, rec.size() * sizeof(ForceAtom)) != hipSuccess ||
        hipMalloc(&op->d_funits, units.size() * sizeof(int)) != hipSuccess ||
        hipMalloc(&op->d_ffun, fun.size() * sizeof(double)) != hipSuccess ||
        hipMalloc(&op->d_fgamma, gam.size() * sizeof(double)) != hipSuccess) {
        for (void **p : {(void **)&op->d_fatoms, (void **)&op->d_funits, (void **)&op->d_ffun,
                         (void **)&op->d_fgamma}) {
            (void)hipFree(*p);
            *p = nullptr;
        }
        return fail(SPARC_E_NOMEM, "allocation of the force tables failed");
    }
    SPARC_HIP(hipMemcpy(op->d_fatoms, rec.data(), rec.size() * sizeof(ForceAtom), hipMemcpyHostToDevice));
    SPARC_HIP(hipMemcpy(op->d_funits, units.data(), units.size() * sizeof(int), hipMemcpyHostToDevice));
    SPARC_HIP(hipMemcpy(op->d_ffun, fun.data(), fun.size() * sizeof(double), hipMemcpyHostToDevice));
    SPARC_HIP(hipMemcpy(op->d_fgamma, gam.data(), gam.size() * sizeof(double), hipMemcpyHostToDevice));
    SPARC_HIP(hipStreamSynchronize(0));  // the caller's stream need not wait for the null stream
    op->force_ready = true;
    return SPARC_OK;
}

// acc[s][t] += contraction of orbital block s (16 columns) with functions 16 t
// .. 16 t + 15 of the box, over this wave's share of its units (groups of 4
// units dealt round-robin to all the waves; lane (i, k) as in gather_accum).
// ROWS: the box of widened rows.  Bits 4 to 7 of a unit's mask are then its
// nodes on the arms, where only F_z (functions fz and up) is not zero by
// definition.  A value there that is not finite must not reach the others
// through a product with their zeros: FAST passes watch for values that are not
// finite (returned), a pass that met one is done again without FAST.
template <typename TI, int NT, int NS, bool ROWS, bool FAST>
__device__ __forceinline__ bool force_pass(const ForceBox &B, const int2 *__restrict__ un,
                                           const double *__restrict__ const (&f)[NT], const TI *const (&y)[NS],
                                           const bool (&ok)[NS], bool small, int step, int wave, int lane,
                                           double (&acc)[NS][NT][4])
{
    typedef TI VY __attribute__((ext_vector_type(kUnit), aligned(sizeof(TI))));
    typedef double VC __attribute__((ext_vector_type(kUnit)));
    const int k = lane >> 4, nu = B.nunits;
    int u = 4 * wave + k;
    int2 qn = un[u < nu ? u : 0];
    TI watch = TI(0);
#pragma unroll 1
    for (int u0 = 4 * wave; u0 < nu; u0 += step) {
        const int2 q = qn;
        const bool in = u < nu;
        const int uc = in ? u : 0;
        u += step;
        qn = un[u < nu ? u : 0];  // the next unit's offset travels while this one's nodes do
        VY yv[NS];
        VC cv[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) cv[t] = *(const VC *)(f[t] + (long long)kUnit * uc);
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            if (!small) {
                yv[s] = *(const VY *)(y[s] + q.x);
            } else {
#pragma unroll
                for (int j = 0; j < kUnit; ++j) yv[s][j] = (q.y >> j) & 1 ? y[s][q.x + j] : TI(0);
            }
        }
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int mask = in && ok[s] ? q.y : 0;
            if (ROWS && FAST) watch += TI(0) * ((yv[s][0] + yv[s][1]) + (yv[s][2] + yv[s][3]));
#pragma unroll
            for (int j = 0; j < kUnit; ++j) {
                double v = (mask >> j) & 1 ? (double)yv[s][j] : 0.0;
                if (ROWS && !FAST && (mask >> (4 + j) & 1) && !__builtin_isfinite(v)) v = 0.0;
#pragma unroll
                for (int t = 0; t < NT; ++t) mfma_16x16x4(v, cv[t][j], acc[s][t]);
            }
        }
    }
    return watch != TI(0);  // 0 times a sum that is not finite is NaN
}

template <typename TI, int NT, int NS, bool ROWS>
__device__ __forceinline__ void force_accum(const ForceBox &B, const int2 *__restrict__ units,
                                            const double *__restrict__ fun, const TI *const (&y)[NS],
                                            const bool (&ok)[NS], bool small, int waves, int wave, int lane, int fz,
                                            double (&acc)[NS][NT][4])
{
    const int i = lane & 15, k = lane >> 4;
    const int2 *un = units + B.unit0;
    const double *f[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int j = 16 * t + i;
        f[t] = fun + B.fun0 + (long long)(j < B.nf ? j : 0) * B.nunits * kUnit;
    }
    const int nu = B.nunits, step = 4 * waves;
    if (nu == 0) return;  // an arm cut off by the walls
    const bool odd = force_pass<TI, NT, NS, ROWS, true>(B, un, f, y, ok, small, step, wave, lane, acc);
    if (!ROWS || !__any(odd)) return;
    // again without the arms' values that are not finite
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[s][t][r] = 0.0;
    (void)force_pass<TI, NT, NS, ROWS, false>(B, un, f, y, ok, small, step, wave, lane, acc);
    // then those values for F_z alone, one tile of sums at a time (few registers)
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            double z[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
            for (int u0 = 4 * wave; u0 < nu; u0 += step) {
                const int e = u0 + k, ec = e < nu ? e : 0;
                const int2 q = un[ec];
                const int arm = e < nu && ok[s] ? q.y >> 4 : 0;
#pragma unroll 1
                for (int j = 0; j < kUnit; ++j) {
                    const double v = arm >> j & 1 ? (double)y[s][q.x + j] : 0.0;
                    mfma_16x16x4(__builtin_isfinite(v) ? 0.0 : v, f[t][(long long)kUnit * ec + j], z);
                }
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[s][t][r] += 16 * t + i >= fz ? z[r] : 0.0;
        }
}

// S_rp(n) below is the contraction of orbital n with function r of projector p.
// Whole (!SPLIT): part[(J ncb + cb) 3 + d] = sum over the workgroup's 16 NS
// orbitals n and the atom's projectors p of occ[n] gamma_p S_0p(n) S_dp(n).
// SPLIT: the workgroup takes share ks of gridDim.z of the units and writes its
// part of S, part[(ks 4 nproj_total + 4 proj0 + r nproj + p) ns + n].
// NT: tiles of 16 functions of the first box (4 nproj <= 16 NT).
template <typename TI, int NT, int NW, int NS, bool SPLIT>
__global__ void __launch_bounds__(64 * NW)
    force_kernel(const TI *__restrict__ psi, long long ld, int ns, int nproj_total,
                 const ForceAtom *__restrict__ atoms, const int2 *__restrict__ units, const double *__restrict__ fun,
                 const double *__restrict__ gamma, const double *__restrict__ occ, int small,
                 double *__restrict__ part)
{
    constexpr int NC = 16 * NS;
    constexpr int G = SPLIT ? 4 : 1;
    __shared__ double S[G][16 * NT][NC];
    __shared__ double red[3][NW];
    const int J = blockIdx.y, cb = blockIdx.x;
    const ForceAtom &F = atoms[J];
    const int c0 = cb * NC, np = F.nproj;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i = lane & 15;
    bool ok[NS];
    const TI *y[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        ok[s] = c0 + 16 * s + i < ns;
        y[s] = psi + (long long)(ok[s] ? c0 + 16 * s + i : c0) * ld;
    }
    // s[rows 16 t + i][columns] (+)= the wave's sums
    auto put = [&](double (*s)[NC], const auto &acc, int rows, bool first) {
#pragma unroll
        for (int b = 0; b < NS; ++b)
#pragma unroll
            for (int t = 0; t < (int)(sizeof(acc[0]) / sizeof(acc[0][0])); ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if (16 * t + i >= rows) continue;
                    double &d = s[16 * t + i][16 * b + acc_row<double>(lane, r)];
                    d = first ? acc[b][t][r] : d + acc[b][t][r];
                }
    };
    if constexpr (SPLIT) {
        // half of the waves take the first box (two copies of S), a quarter each
        // arm (a copy each): one pass over the units, NW / 4 rounds of sums
        constexpr int NB = NW / 2, NA = NW / 4;
        const int box = wave < NB ? 0 : 1 + (wave - NB) / NA, w = box ? wave % NA : wave, parts = gridDim.z;
        double acc[NS][NT][4] = {}, arm[NS][1][4] = {};
        if (box == 0)
            force_accum<TI, NT, NS, true>(F.box[0], units, fun, y, ok, small != 0, NB * parts, NB * blockIdx.z + w, lane,
                                          3 * np, acc);
        else
            force_accum<TI, 1, NS, false>(F.box[box], units, fun, y, ok, small != 0, NA * parts, NA * blockIdx.z + w, lane,
                                          0, arm);
        for (int r = 0; r < NA; ++r) {
            if (box == 0 && w / 2 == r) put(S[w & 1], acc, 16 * NT, r == 0);
            if (box != 0 && w == r) put(S[1 + box] + box * np, arm, np, r == 0);
            __syncthreads();
        }
        for (int e = threadIdx.x; e < 4 * np * NC; e += 64 * NW) {
            const int j = e / NC, c = e % NC, r = j / np;
            double v = S[0][j][c] + S[1][j][c];
            if (r == 1 || r == 2) v += S[1 + r][j][c];
            if (c0 + c < ns) part[((long long)blockIdx.z * 4 * nproj_total + 4 * F.proj0 + j) * ns + c0 + c] = v;
        }
        return;
    }
    {
        double acc[NS][NT][4] = {};
        force_accum<TI, NT, NS, true>(F.box[0], units, fun, y, ok, small != 0, NW, wave, lane, 3 * np, acc);
        for (int w = 0; w < NW; ++w) {
            if (wave == w) put(S[0], acc, 16 * NT, w == 0);
            __syncthreads();
        }
    }
#pragma unroll 1
    for (int k = 1; k < 3; ++k) {
        double acc[NS][1][4] = {};
        force_accum<TI, 1, NS, false>(F.box[k], units, fun, y, ok, small != 0, NW, wave, lane, 0, acc);
        for (int w = 0; w < NW; ++w) {
            if (wave == w) put(S[0] + k * np, acc, np, false);
            __syncthreads();
        }
    }
    const int c = threadIdx.x % NC;
    double v[3] = {0.0, 0.0, 0.0};
    if (c0 + c < ns) {
        for (int p = threadIdx.x / NC; p < np; p += 64 * NW / NC) {
            const double gy = gamma[F.proj0 + p] * S[0][p][c];
#pragma unroll
            for (int d = 0; d < 3; ++d) v[d] += gy * S[0][(1 + d) * np + p][c];
        }
        const double g = occ[c0 + c];
#pragma unroll
        for (int d = 0; d < 3; ++d) v[d] *= g;
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        for (int off = 32; off > 0; off >>= 1) v[d] += __shfl_xor(v[d], off);
        if (lane == 0) red[d][wave] = v[d];
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        double f = 0.0;
#pragma unroll
        for (int w = 0; w < NW; ++w) f += red[threadIdx.x][w];
        part[((long long)J * gridDim.x + cb) * 3 + threadIdx.x] = f;
    }
}

// force[e] = scale * sum over the orbital blocks, in order; e = 3 J + d
__global__ void __launch_bounds__(64) force_sum_kernel(const double *__restrict__ part, int ncb, int n3, double scale,
                                                          double *__restrict__ force)
{
    const int e = blockIdx.x * 64 + threadIdx.x;
    if (e >= n3) return;
    double v = 0.0;
#pragma unroll 8
    for (int b = 0; b < ncb; ++b) v += part[((long long)(e / 3) * ncb + b) * 3 + e % 3];
    force[e] = scale * v;
}

constexpr int kFinishThreads = 1024;

// one workgroup per atom: f[3J + d] = scale * sum_n occ[n] sum_p gamma_p S_0p(n) S_dp(n),
// S the sum of the parts in order; the (projector, orbital) pairs are dealt to
// the threads, whose sums meet in a fixed butterfly and wave order
__global__ void __launch_bounds__(kFinishThreads) force_finish_kernel(const double *__restrict__ part, int parts, int nproj_total,
                                                           int ns, const ForceAtom *__restrict__ atoms,
                                                           const double *__restrict__ gamma,
                                                           const double *__restrict__ occ, double scale,
                                                           double *__restrict__ force)
{
    const int np = atoms[blockIdx.x].nproj, proj0 = atoms[blockIdx.x].proj0;
    const long long split = 4LL * nproj_total * ns;
    double acc[3] = {0.0, 0.0, 0.0};
    for (long long e = threadIdx.x; e < (long long)np * ns; e += kFinishThreads) {
        const int p = (int)(e / ns), n = (int)(e - (long long)p * ns);
        const double *q = part + (4LL * proj0 + p) * ns + n;
        double S[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
        for (int k = 0; k < parts; ++k)
#pragma unroll
            for (int r = 0; r < 4; ++r) S[r] += q[k * split + (long long)r * np * ns];
        const double gy = occ[n] * (gamma[proj0 + p] * S[0]);
#pragma unroll
        for (int d = 0; d < 3; ++d) acc[d] += gy * S[1 + d];
    }
    __shared__ double red[3][kFinishThreads / 64];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        double v = acc[d];
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
        if ((threadIdx.x & 63) == 0) red[d][threadIdx.x >> 6] = v;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        double v = 0.0;
#pragma unroll
        for (int w = 0; w < kFinishThreads / 64; ++w) v += red[threadIdx.x][w];
        force[3 * blockIdx.x + threadIdx.x] = scale * v;
    }
}

template <typename TI, int NW, int NS, bool SPLIT>
void launch_force(const sparc_op *op, const TI *psi, long long ld, int ns, const double *occ, int parts, double *part,
                  double *force, hipStream_t s)
{
    const int ncb = (ns + 16 * NS - 1) / (16 * NS), small = op->nd < kUnit;
    const int2 *units = (const int2 *)op->d_funits;
    const double *fun = op->d_ffun, *gamma = op->d_fgamma;
    const double h3 = op->h * op->h * op->h, scale = -4.0 * h3 * h3;
    for (int J = 0; J < op->natoms; J += 65535) {
        const ForceAtom *atoms = (const ForceAtom *)op->d_fatoms + J;
        const dim3 grid(ncb, std::min(op->natoms - J, 65535), parts), b(64 * NW);
        double *out = SPLIT ? part : part + 3LL * J * ncb;
#define SPARC_FORCE(N)                                                                                               \
    hipLaunchKernelGGL((force_kernel<TI, N, NW, NS, SPLIT>), grid, b, 0, s, psi, ld, ns, op->nproj_total, atoms, units, \
                       fun, gamma, occ, small, out)
        switch ((4 * op->max_nproj + 15) / 16) {
            case 1: SPARC_FORCE(1); break;
            case 2: SPARC_FORCE(2); break;
            case 3: SPARC_FORCE(3); break;
            default: SPARC_FORCE(4); break;
        }
#undef SPARC_FORCE
    }
    if (SPLIT)
        hipLaunchKernelGGL(force_finish_kernel, dim3(op->natoms), dim3(kFinishThreads), 0, s, part, parts,
                           op->nproj_total, ns, (const ForceAtom *)op->d_fatoms, gamma, occ, scale, force);
    else
        hipLaunchKernelGGL(force_sum_kernel, dim3((3 * op->natoms + 63) / 64), dim3(64), 0, s, part, ncb,
                           3 * op->natoms, scale, force);
}

// Whole units lists per workgroup once the chip is full of them.  Measured,
// FP32, whole against 4 parts: 512 workgroups (128 atoms x 100 orbitals) 482
// against 383 us, 589 (31 x 600) 510 against 488, 1024 (FP64, 128 x 240) 944
// against 999, 2432 (128 x 600, 9 projectors) 2257 against 2453.
bool force_whole(const sparc_op *op, int ns) { return (long long)op->natoms * ((ns + 31) / 32) >= 1024; }

// Parts of the units of a split launch: 16 where an atom and 16 orbitals make
// fewer than 32 workgroups (96^3, 16 atoms x 12 orbitals: 15.2 us, with 4
// parts 23.6), else 4 (48^3, 2 atoms x 300 orbitals: 34, with 16 parts 54 us).
constexpr int kMinParts = 4, kMaxParts = 16;
int force_parts(const sparc_op *op, int ns)
{
    return (long long)op->natoms * ((ns + 15) / 16) < 32 ? kMaxParts : kMinParts;
}

// the partial sums; a whole launch writes natoms x orbital blocks x 3 values of them
size_t force_part_bytes(const sparc_op *op, int ns, int parts)
{
    return (size_t)parts * 4 * op->nproj_total * ns * sizeof(double);
}

template <typename TI>
void force_any(const sparc_op *op, const TI *psi, long long ld, int ns, const double *occ, double *part,
               int parts, double *force, hipStream_t s)
{
    if (force_whole(op, ns))
        launch_force<TI, 4, 2, false>(op, psi, ld, ns, occ, 1, part, force, s);
    else
        launch_force<TI, 8, 1, true>(op, psi, ld, ns, occ, parts, part, force, s);
}

}  // namespace
}  // namespace sparc

using namespace sparc;

extern "C" size_t sparc_force_workspace_bytes(const sparc_op *op, int32_t ns)
{
    if (!op || ns < 1) return 0;
    return std::max<size_t>(force_part_bytes(op, ns, force_parts(op, ns)), 256);
}

extern "C" int sparc_nonlocal_force(const sparc_op *op, int32_t dtype, const void *psi, int64_t ld, int32_t ns,
                                    const double *occ, double *force, void *ws, size_t ws_bytes, void *stream)
{
    if (!op || !psi || !occ || (op->natoms > 0 && !force) || (dtype != SPARC_F64 && dtype != SPARC_F32))
        return fail(SPARC_E_ARG, "bad arguments");
    if (ns < 1 || ld < op->nd) return fail(SPARC_E_SHAPE, "ns < 1 or ld < N_d");
    if ((ns + 15) / 16 > 65535) return fail(SPARC_E_SHAPE, "too many columns for one launch");
    if (op->natoms == 0) return SPARC_OK;
    const size_t need = force_part_bytes(op, ns, kMinParts);
    if (!ws || ws_bytes < need) return fail(SPARC_E_WORKSPACE, "workspace missing or too small");
    const size_t es = elem_size(dtype);
    const char *p0 = (const char *)psi, *p1 = p0 + ((size_t)(ns - 1) * ld + op->nd) * es;
    const char *w0 = (const char *)ws;
    const char *f0 = (const char *)force, *f1 = f0 + (size_t)op->natoms * 3 * sizeof(double);
    auto overlap = [&](size_t bytes) {
        const char *w1 = w0 + bytes;
        return (w0 < p1 && p0 < w1) || (f0 < w1 && w0 < f1);
    };
    if (overlap(need) || (f0 < p1 && p0 < f1)) return fail(SPARC_E_ALIAS, "psi, the workspace and the forces overlap");
    // a workspace without room for the parts this size is best split into gets the fewest
    int parts = force_parts(op, ns);
    const size_t room = force_part_bytes(op, ns, parts);
    if (ws_bytes < room || overlap(room)) parts = kMinParts;
    {
        std::lock_guard<std::mutex> lk(op->force_mu);
        if (!op->force_ready) {
            int st = build_force_tables(op);
            if (st) return st;
        }
    }
    TraceRange trace("sparc_nonlocal_force");
    hipStream_t s = (hipStream_t)stream;
    ProfScope prof(5, s);
    if (dtype == SPARC_F64)
        force_any(op, (const double *)psi, ld, ns, occ, (double *)ws, parts, force, s);
    else
        force_any(op, (const float *)psi, ld, ns, occ, (double *)ws, parts, force, s);
    SPARC_HIP(hipGetLastError());
    return SPARC_OK;
}
