// Device side of the nonlocal gather and scatter (see nonlocal.hip for the
// design); shared by the standalone launches and the batched persistent kernel.
#pragma once

#include "internal.hpp"

namespace sparc {

// The gather reads an atom's cube as units of 4 consecutive grid nodes (built
// at operator creation): x is the grid index of the unit's first node, bit j
// of y says whether node j belongs to the cube (a unit at the edge of a row
// also covers nodes outside it).
constexpr int kUnit = 4;

// TI: storage type of Y (FP32 blocks may be projected in FP64)
template <typename T, typename TI = T>
struct GatherArgs {
    const TI *Y;
    long long ldy;
    int ns;
    int nproj_total;
    int small;           // fewer than kUnit grid nodes: Y is read node by node
    const AtomDev *atoms;
    const int2 *units;   // per atom from atom.unit0
    const T *chiu;       // per atom from atom.chiu0: [projector][unit][kUnit], zero off the cube
    const int *box_off;  // grid index of every cube node, per atom from atom.box0
    const T *chi;        // per atom from atom.chi0: [projector][cube node]
    T *part;             // [kGatherSplit (1: gather_whole_kernel)][nproj_total][ns] projections
};

__device__ inline void mfma_16x16x4(const double a, const double b, double (&acc)[4])
{
    typedef double v4d __attribute__((ext_vector_type(4)));
    v4d c = {acc[0], acc[1], acc[2], acc[3]};
    c = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    acc[0] = c[0];
    acc[1] = c[1];
    acc[2] = c[2];
    acc[3] = c[3];
}

__device__ inline void mfma_16x16x4(const float a, const float b, float (&acc)[4])
{
    typedef float v4f __attribute__((ext_vector_type(4)));
    v4f c = {acc[0], acc[1], acc[2], acc[3]};
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    acc[0] = c[0];
    acc[1] = c[1];
    acc[2] = c[2];
    acc[3] = c[3];
}

// accumulator row held by register r of this lane
template <typename T>
__device__ inline int acc_row(int lane, int r)
{
    if constexpr (sizeof(T) == 8)
        return (lane >> 4) + 4 * r;
    else
        return 4 * (lane >> 4) + r;
}

// An atom's units are cut into 4 kGatherSplit segments of whole groups of 4
// units, each summed by one wave; the order of the sums depends on nothing
// else, so a projection has the same bits in every launch shape.
__device__ __forceinline__ int gather_segment(int nunits)
{
    constexpr int S = 4 * kGatherSplit;
    return ((nunits + S - 1) / S + 3) / 4 * 4;
}

// acc += chi^T Y over units [u0, u1) for 16 columns x 16 projectors: lane
// (i, k) loads the 16-byte units u0 + k, u0 + k + 4, ... of column i and of
// projector i; the j-th matrix instruction of a load takes node j of the four
// units (node j of unit k is contraction index k on both operands).
template <typename T, typename TI, int UNROLL>
__device__ __forceinline__ void gather_accum(const GatherArgs<T, TI> &g, const TI *y, const T *ch, const int2 *units,
                                             int u0, int u1, bool col_ok, int k, T (&acc)[4])
{
    typedef TI VY __attribute__((ext_vector_type(kUnit), aligned(sizeof(TI))));
    typedef T VC __attribute__((ext_vector_type(kUnit)));
#pragma unroll 1
    for (int base = u0; base < u1; base += 4 * UNROLL) {
        int2 un[UNROLL];
        VY yv[UNROLL];
        VC cv[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const int e = base + 4 * u + k;
            un[u] = units[e < u1 ? e : u0];
            if (e >= u1 || !col_ok) un[u].y = 0;
        }
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const int e = base + 4 * u + k;
            cv[u] = *(const VC *)(ch + (long long)kUnit * (e < u1 ? e : u0));
            if (!g.small) {
                yv[u] = *(const VY *)(y + un[u].x);
            } else {
#pragma unroll
                for (int j = 0; j < kUnit; ++j) yv[u][j] = (un[u].y >> j) & 1 ? y[un[u].x + j] : TI(0);
            }
        }
#pragma unroll
        for (int u = 0; u < UNROLL; ++u)
#pragma unroll
            for (int j = 0; j < kUnit; ++j)
                mfma_16x16x4((un[u].y >> j) & 1 ? (T)yv[u][j] : T(0), (T)cv[u][j], acc);
    }
}

// tid: this thread's index within the 256 threads (4 waves) that run the
// item; the item has one workgroup barrier.  Two units per lane are loaded
// together (more take registers, so waves in flight: 96^3 x 64 FP64 with 16
// cubes 13.0 us with 2, 14.4 with 4, 16.0 with 8; FP32 9.8, 10.7, 11.2)
template <typename T, typename TI = T>
__device__ __forceinline__ void gather_units(const GatherArgs<T, TI> &g, int atom, int cb, int ks, T (*tile)[16][16],
                                            int tid)
{
    const int c0 = cb * 16;
    const AtomDev A = g.atoms[atom];
    const int seg = gather_segment(A.nunits);
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int i = lane & 15;
    const int col = c0 + i;
    const bool col_ok = col < g.ns;
    const int u0 = min(A.nunits, (4 * ks + wave) * seg), u1 = min(A.nunits, u0 + seg);
    T acc[4] = {T(0), T(0), T(0), T(0)};
    gather_accum<T, TI, 2>(g, g.Y + (long long)(col_ok ? col : 0) * g.ldy,
                           g.chiu + A.chiu0 + (long long)(i < A.nproj ? i : 0) * A.nunits * kUnit, g.units + A.unit0, u0,
                           u1, col_ok, lane >> 4, acc);
#pragma unroll
    for (int r = 0; r < 4; ++r) tile[wave][acc_row<T>(lane, r)][lane & 15] = acc[r];
    __syncthreads();
    const int row = tid >> 4, pj = tid & 15;
    const int cc = c0 + row;
    if (cc < g.ns && pj < A.nproj) {
        const T s = ((tile[0][row][pj] + tile[1][row][pj]) + tile[2][row][pj]) + tile[3][row][pj];
        g.part[((long long)ks * g.nproj_total + A.proj0 + pj) * g.ns + cc] = s;
    }
}

constexpr int kGatherUnroll = 8;  // groups of 4 points per wave per batch

// One split of an atom's cube node by node (FP64 blocks).  An FP64 node is half
// of a 16-byte load already, and units of 4 would pad the rows of 14 to 15
// nodes by a quarter more matrix instructions, which are on the critical path
// of the small FP64 launches: by units a filter step of 48^3 x 11 took 17.7
// instead of 17.0 us, H of one 148 x 132 x 145 column 32.6 instead of 31.1 us;
// 96^3 x 64 the same 13 us.
// tid: this thread's index within the 256 threads (4 waves) that run the
// item; the item has one workgroup barrier
template <typename T, typename TI = T>
__device__ __forceinline__ void gather_nodes(const GatherArgs<T, TI> &g, int atom, int cb, int ks, T (*tile)[16][16],
                                            int tid)
{
    const int c0 = cb * 16;
    const AtomDev A = g.atoms[atom];
    const int nbox = A.ext[0] * A.ext[1] * A.ext[2];
    const int chunk = (nbox + kGatherSplit - 1) / kGatherSplit;
    const int k0 = min(nbox, ks * chunk);
    const int k1 = min(nbox, k0 + chunk);
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int i = lane & 15;
    const int k = lane >> 4;
    const int col = c0 + i;
    const bool col_ok = col < g.ns;
    const bool proj_ok = i < A.nproj;
    const TI *y = g.Y + (long long)(col_ok ? col : 0) * g.ldy;
    const T *ch = g.chi + A.chi0 + (long long)(proj_ok ? i : 0) * nbox;
    const int *boff = g.box_off + A.box0;

    T acc[4] = {T(0), T(0), T(0), T(0)};
    constexpr int BATCH = 4 * kGatherUnroll;
    for (int base = k0 + wave * BATCH; base < k1; base += 4 * BATCH) {
        int off[kGatherUnroll];
        T av[kGatherUnroll], bv[kGatherUnroll];
#pragma unroll
        for (int u = 0; u < kGatherUnroll; ++u) {
            const int pt = base + 4 * u + k;
            off[u] = boff[pt < k1 ? pt : k0];
        }
#pragma unroll
        for (int u = 0; u < kGatherUnroll; ++u) {
            const int pt = base + 4 * u + k;
            const bool ok = pt < k1;
            const T yv = (T)y[off[u]];
            const T cv = ch[ok ? pt : k0];
            av[u] = (ok && col_ok) ? yv : T(0);
            bv[u] = (ok && proj_ok) ? cv : T(0);
        }
#pragma unroll
        for (int u = 0; u < kGatherUnroll; ++u) mfma_16x16x4(av[u], bv[u], acc);
    }

#pragma unroll
    for (int r = 0; r < 4; ++r) tile[wave][acc_row<T>(lane, r)][lane & 15] = acc[r];
    __syncthreads();
    const int row = tid >> 4, pj = tid & 15;
    const int cc = c0 + row;
    if (cc < g.ns && pj < A.nproj) {
        const T s = ((tile[0][row][pj] + tile[1][row][pj]) + tile[2][row][pj]) + tile[3][row][pj];
        g.part[((long long)ks * g.nproj_total + A.proj0 + pj) * g.ns + cc] = s;
    }
}

// one item of the gather: FP32 storage by units, FP64 node by node
template <typename T, typename TI = T>
__device__ __forceinline__ void gather_item(const GatherArgs<T, TI> &g, int atom, int cb, int ks, T (*tile)[16][16],
                                            int tid)
{
    if constexpr (sizeof(TI) == 4)
        gather_units<T, TI>(g, atom, cb, ks, tile, tid);
    else
        gather_nodes<T, TI>(g, atom, cb, ks, tile, tid);
}

// all kGatherSplit items of (atom, cb) in one 256-thread workgroup, their
// partials summed in split order as the consumers of gather_item's partials
// sum them: part holds the finished projections.  tile: 16 tiles
template <typename T, typename TI = T>
__device__ __forceinline__ void gather_whole(const GatherArgs<T, TI> &g, int atom, int cb, T (*tile)[4][16][16])
{
    static_assert(kGatherSplit % 4 == 0, "tiles go through LDS four splits at a time");
    const int c0 = cb * 16, tid = threadIdx.x;
    const AtomDev A = g.atoms[atom];
    const int seg = gather_segment(A.nunits);
    const int lane = tid & 63, wave = tid >> 6, i = lane & 15;
    const int col = c0 + i;
    const bool col_ok = col < g.ns;
    const TI *y = g.Y + (long long)(col_ok ? col : 0) * g.ldy;
    const T *ch = g.chiu + A.chiu0 + (long long)(i < A.nproj ? i : 0) * A.nunits * kUnit;
    const int row = tid >> 4, pj = tid & 15;
    T s = T(0);
#pragma unroll 1
    for (int q0 = 0; q0 < kGatherSplit; q0 += 4) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int u0 = min(A.nunits, (4 * (q0 + q) + wave) * seg), u1 = min(A.nunits, u0 + seg);
            T acc[4] = {T(0), T(0), T(0), T(0)};
            gather_accum<T, TI, 4>(g, y, ch, g.units + A.unit0, u0, u1, col_ok, lane >> 4, acc);
#pragma unroll
            for (int r = 0; r < 4; ++r) tile[q][wave][acc_row<T>(lane, r)][lane & 15] = acc[r];
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 4; ++q)
            s += ((tile[q][0][row][pj] + tile[q][1][row][pj]) + tile[q][2][row][pj]) + tile[q][3][row][pj];
        __syncthreads();
    }
    if (c0 + row < g.ns && pj < A.nproj) g.part[((long long)A.proj0 + pj) * g.ns + c0 + row] = s;
}

constexpr int kScatterCols = 8;  // columns per scatter item of the batched kernel

template <typename T>
struct ScatterArgs {
    T *out;
    long long ldo;
    int ns;
    int nproj_total;
    const int *blk_pt;     // nblk + 1 node offsets
    const int *blk_at;     // nblk + 1 offsets into blk_atoms
    const int *blk_atoms;  // atoms touched by each block (slot order)
    const int *pts;        // unique grid nodes covered by a cube
    const int *ent_off;    // npts + 1 offsets into ent
    const int4 *ent;       // (chi index of projector 0, cube size, slot, nproj)
    const AtomDev *atoms;
    const T *chi;
    const T *hg;           // h^3 gamma per global projector
    const T *part;         // [NP][nproj_total][ns]
    T alpha;
};

// One node block b (at most 256 nodes) and NC columns from cg * NC.  NP: parts
// of the projections (kGatherSplit, or 1: finished).  gl: the
// block's table h^3 gamma S, [slot][npm][NC] (npm >= every atom's projector
// count).  The out values of all NC columns are requested before the table
// is built, so their latency overlaps it.  Per node and column the sum runs
// over the node's entries and projectors in table order whatever NC is, so
// every column count gives the same bits.
template <typename T, int NC, int NP = kGatherSplit>
__device__ __forceinline__ void scatter_item(const ScatterArgs<T> &s, int b, int cg, T *gl, int npm)
{
    const int c0 = cg * NC;
    const int a0 = s.blk_at[b];
    const int na = s.blk_at[b + 1] - a0;
    const long long split = (long long)s.nproj_total * s.ns;
    const int pi = s.blk_pt[b] + threadIdx.x;
    const bool own = pi < s.blk_pt[b + 1];
    int gpt = 0, e0 = 0, e1 = 0;
    T cur[NC];
#pragma unroll
    for (int cc = 0; cc < NC; ++cc) cur[cc] = T(0);
    if (own) {
        gpt = s.pts[pi];
        e0 = s.ent_off[pi];
        e1 = s.ent_off[pi + 1];
#pragma unroll
        for (int cc = 0; cc < NC; ++cc)
            if (c0 + cc < s.ns) cur[cc] = s.out[(long long)(c0 + cc) * s.ldo + gpt];
    }
    for (int idx = threadIdx.x; idx < na * npm * NC; idx += 256) {
        const int slot = idx / (npm * NC);
        const int p = (idx / NC) % npm;
        const int cc = idx % NC;
        const AtomDev A = s.atoms[s.blk_atoms[a0 + slot]];
        T v = T(0);
        if (p < A.nproj && c0 + cc < s.ns) {
            const long long pg = A.proj0 + p;
            T sum = T(0);
#pragma unroll
            for (int q = 0; q < NP; ++q) sum += s.part[q * split + pg * s.ns + c0 + cc];
            v = s.hg[pg] * sum;
        }
        gl[idx] = v;
    }
    __syncthreads();
    if (!own) return;
    T acc[NC];
#pragma unroll
    for (int cc = 0; cc < NC; ++cc) acc[cc] = T(0);
    for (int e = e0; e < e1; ++e) {
        const int4 en = s.ent[e];
        for (int p = 0; p < en.w; ++p) {
            const T cv = s.chi[en.x + (long long)p * en.y];
            const T *row = gl + (en.z * npm + p) * NC;
#pragma unroll
            for (int cc = 0; cc < NC; ++cc) acc[cc] += cv * row[cc];
        }
    }
#pragma unroll
    for (int cc = 0; cc < NC; ++cc)
        if (c0 + cc < s.ns) s.out[(long long)(c0 + cc) * s.ldo + gpt] = cur[cc] + s.alpha * acc[cc];
}

}  // namespace sparc
