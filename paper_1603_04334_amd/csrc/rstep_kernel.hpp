// Device side of the row-pair step: the vector step (stencil, local potential
// and Chebyshev recurrence in one pass over an orbital block, see fstep.hip)
// with two consecutive y rows per lane and a patch whose extents are chosen at
// run time to fit the grid.
//
// Why two rows: with one 16-byte unit per lane the step launch spends its time
// in LDS reads and FP32 arithmetic that a workgroup's waves run in the same
// phase, not in HBM.  A lane that owns rows y and y + 1 reads the 12 rows
// y - 6 .. y - 1 and y + 2 .. y + 7 once for both, 6 units per row instead of
// 12 (9 instead of 15 reads of 16 bytes per FP32 unit with the z window), at
// the price of two register queues: 8 waves of up to 256 registers per CU.
// One load stage (one plane ahead) is enough, a plane of such a patch takes
// longer than a memory access.
//
// What bounds it now: at 160^3 x 600 FP32 the launch without projectors takes
// 5.80 to 5.85 ms (6.96 ms before, 32 x 32 patches; 5.71 ms with x in 4 chunks
// and groups of 4 columns), 29.5 GB at 5.09 TB/s; a kernel that
// only walks the same three arrays in the same order of planes takes 5.78 ms
// (a linear walk of them 4.61 ms), and leaving out V_eff, the halo and the LDS
// reads together gains 4 %.  The order of the walk is what is left.
#pragma once

#include "fstep_kernel.hpp"

namespace sparc {

template <typename T>
struct RStepArgs {
    const T *yk;
    const T *yprev;
    T *out;
    const T *veff;
    long long ldk, ldp, ldo;
    int n1, n2, n3;
    int tz, ty, lpr;  // patch extents (tz a multiple of the unit, ty even), lanes per patch row
    int tiles_y, tiles_z, nchunks, chunk_x;
    int nblocks;
    int ns, cgroup;
    int zhalo;         // the patch is narrower than a grid row: it has a z halo
    T c0;              // -3 w_0
    T cp[kMaxRadius];  // -1/2 w_p
    T alpha, beta, shift;
};

// PITCH: elements per LDS row.  NH: halo units per lane and plane.  RAG: the
// nodes by which a row falls short of whole units (0: none).  The lane of the
// cut unit loads the last VZ nodes of the row, so that every load stays inside
// the row, and moves them to their places in the unit (zeros past the row end):
// LDS and the queues hold whole aligned units whatever the row.
template <typename T, int PITCH, int NH, bool PREV, bool STREAM, int RAG>
struct RStep {
    static constexpr int R = kMaxRadius;
    static constexpr int VZ = VecTraits<T>::N;
    using V = typename VecTraits<T>::V;
    typedef T VH __attribute__((ext_vector_type(VZ / 2)));
    static constexpr int PADZ = (R + VZ - 1) / VZ * VZ;
    static constexpr int ZU = PADZ / VZ;
    static constexpr int QL = 2 * R + 1;
    static constexpr int WU = 2 * ZU + 1;
    static_assert(PITCH % VZ == 0, "whole units per LDS row");

    const RStepArgs<T> &a;
    const T *yk;
    const T *yp;
    T *out;
    long long P;
    T *L0;            // the lane's first own value in LDS buffer 0
    T *Lh[NH];        // its halo units there (null: none)
    int bufe;         // elements per LDS buffer
    bool own;         // lane of the patch (the others only load halo units)
    bool cut;         // RAG: the lane's unit is cut by the row end
    bool hcut[NH];    // RAG: so is this halo unit
    unsigned pofs[2];   // in-plane byte offsets of the two units, or kOutside
    unsigned hofs[NH];
    V q[2][QL];
    V sh[NH], sq[2], sv[2], sp[2];  // the load stage

    __device__ RStep(const RStepArgs<T> &args) : a(args) {}

    template <int Q>
    static constexpr int slot(int d) { return (Q + d) % QL; }

    static __device__ __forceinline__ V place(const V &v, bool c) { return place_unit<T, RAG>(v, c); }

    __device__ __forceinline__ void load_head(int t)
    {
        const auto rk = plane_rsrc(yk, t, a.n1, P);
#pragma unroll
        for (int i = 0; i < NH; ++i) sh[i] = vload<T, 0>(rk, hofs[i]);
        const auto rq = plane_rsrc(yk, t + R, a.n1, P);
#pragma unroll
        for (int r = 0; r < 2; ++r) sq[r] = vload<T, 0>(rq, pofs[r]);
    }

    __device__ __forceinline__ void load_point(int t)
    {
        const auto rv = plane_rsrc(a.veff, t, a.n1, P);
#pragma unroll
        for (int r = 0; r < 2; ++r) sv[r] = vload<T, 0>(rv, pofs[r]);
        if constexpr (PREV) {
            const auto rp = plane_rsrc(yp, t, a.n1, P);
#pragma unroll
            for (int r = 0; r < 2; ++r) sp[r] = vload<T, STREAM ? kNonTemporal : 0>(rp, pofs[r]);
        }
    }

    // the z window of row r: values [-PADZ, PADZ + VZ) around the lane's unit,
    // the centre from registers, of the edge units only the used aligned half
    __device__ __forceinline__ void window(const T *row, const V &cen, T (&w)[WU * VZ])
    {
        constexpr int WLO = PADZ - R, WHI = PADZ + VZ - 1 + R;
#pragma unroll
        for (int u = 0; u < WU; ++u) {
            const int u0 = u * VZ, u1 = u0 + VZ - 1;
            const int b0 = u0 > WLO ? u0 : WLO, b1 = u1 < WHI ? u1 : WHI;
            if (u == ZU) {
#pragma unroll
                for (int j = 0; j < VZ; ++j) w[u0 + j] = cen[j];
            } else if (b0 == u0 && b1 == u1) {
                const V t = *(const V *)&row[u0 - PADZ];
#pragma unroll
                for (int j = 0; j < VZ; ++j) w[u0 + j] = t[j];
            } else if (b0 <= b1) {
                constexpr int H = VZ / 2;
                const int h0 = (b0 - u0) / H * H;
                const VH t = *(const VH *)&row[u0 + h0 - PADZ];
#pragma unroll
                for (int j = 0; j < H; ++j) w[u0 + h0 + j] = t[j];
            }
        }
    }

    template <int Q>
    __device__ __forceinline__ void plane(int x, int buf)
    {
        T *L = L0 + buf;
#pragma unroll
        for (int r = 0; r < 2; ++r) q[r][slot<Q>(2 * R)] = place(sq[r], cut);
        if (own) {
            *(V *)&L[0] = q[0][slot<Q>(R)];
            *(V *)&L[PITCH] = q[1][slot<Q>(R)];
        }
#pragma unroll
        for (int i = 0; i < NH; ++i)
            if (Lh[i]) *(V *)(Lh[i] + buf) = place(sh[i], hcut[i]);
        __syncthreads();

        load_head(x + 1);

        const V cen0 = q[0][slot<Q>(R)], cen1 = q[1][slot<Q>(R)];
        T w0[WU * VZ], w1[WU * VZ], acc0[VZ], acc1[VZ];
        window(L, cen0, w0);
        window(L + PITCH, cen1, w1);
#pragma unroll
        for (int j = 0; j < VZ; ++j) {
            acc0[j] = a.c0 * cen0[j];
            acc1[j] = a.c0 * cen1[j];
        }
        // rows y - p and y + 1 + p are new at distance p; y + p and y + 1 - p
        // were read at p - 1
        V lo1 = cen0, hi0 = cen1;
#pragma unroll
        for (int p = 1; p <= R; ++p) {
            const V lo = *(const V *)&L[-p * PITCH];
            const V hi = *(const V *)&L[(1 + p) * PITCH];
#pragma unroll
            for (int j = 0; j < VZ; ++j) {
                const T s0 = (q[0][slot<Q>(R - p)][j] + q[0][slot<Q>(R + p)][j]) + (lo[j] + hi0[j]) +
                             (w0[PADZ + j - p] + w0[PADZ + j + p]);
                acc0[j] += a.cp[p - 1] * s0;
                const T s1 = (q[1][slot<Q>(R - p)][j] + q[1][slot<Q>(R + p)][j]) + (lo1[j] + hi[j]) +
                             (w1[PADZ + j - p] + w1[PADZ + j + p]);
                acc1[j] += a.cp[p - 1] * s1;
            }
            lo1 = lo;
            hi0 = hi;
        }
        V r0, r1;
        const V v0 = place(sv[0], cut), v1 = place(sv[1], cut);
        V p0, p1;
        if constexpr (PREV) {
            p0 = place(sp[0], cut);
            p1 = place(sp[1], cut);
        }
#pragma unroll
        for (int j = 0; j < VZ; ++j) {
            acc0[j] += (v0[j] - a.shift) * cen0[j];
            acc1[j] += (v1[j] - a.shift) * cen1[j];
            T u0 = a.alpha * acc0[j], u1 = a.alpha * acc1[j];
            if constexpr (PREV) {
                u0 -= a.beta * p0[j];
                u1 -= a.beta * p1[j];
            }
            r0[j] = u0;
            r1[j] = u1;
        }
        const auto ro = plane_rsrc((const T *)out, x, a.n1, P);
        constexpr int AUX = STREAM ? kNonTemporal : 0;
        if (RAG > 0 && cut) {
            // pofs points at the nodes loaded, RAG nodes before the unit
#pragma unroll
            for (int j = 0; j + RAG < VZ; ++j) {
                buf_store<T, AUX>(r0[j], ro, pofs[0] + (j + RAG) * (unsigned)sizeof(T));
                buf_store<T, AUX>(r1[j], ro, pofs[1] + (j + RAG) * (unsigned)sizeof(T));
            }
        } else {
            vstore<T, AUX>(r0, ro, pofs[0]);
            vstore<T, AUX>(r1, ro, pofs[1]);
        }
        load_point(x + 1);
    }

    template <int U>
    __device__ __forceinline__ void run_block(int x0, int xend, int buf)
    {
        if constexpr (U < QL) {
            if (x0 + U >= xend) return;
            plane<U>(x0 + U, buf);
            run_block<U + 1>(x0, xend, bufe - buf);
        }
    }

    // in-plane byte offset of the unit at (gy, gz); c: cut by the row end
    __device__ __forceinline__ unsigned unit_ofs(int gy, int gz, bool ok, bool &c) const
    {
        c = false;
        if (!ok || gy < 0 || gy >= a.n2 || gz < 0 || gz >= a.n3) return kOutside;
        if constexpr (RAG > 0) c = gz + VZ > a.n3;
        return (unsigned)(gy * a.n3 + gz - (c ? RAG : 0)) * (unsigned)sizeof(T);
    }

    __device__ __forceinline__ void run(int wg, T *lds)
    {
        const int nb = a.nblocks;
        const int xcd = wg & 7;
        int t = xcd * (nb >> 3) + min(xcd, nb & 7) + (wg >> 3);
        const int cg = t % a.cgroup;
        t /= a.cgroup;
        const int tzi = t % a.tiles_z;
        t /= a.tiles_z;
        const int tyi = t % a.tiles_y;
        t /= a.tiles_y;
        const int chunk = t % a.nchunks;
        const int col = (t / a.nchunks) * a.cgroup + cg;
        if (col >= a.ns) return;  // the padding of the last column group

        const int tid = threadIdx.x, nt = blockDim.x;
        const int lp = tid / a.lpr, lz = tid - lp * a.lpr;
        const int z0 = tzi * a.tz, y0 = tyi * a.ty;
        P = (long long)a.n2 * a.n3;
        yk = a.yk + (size_t)col * a.ldk;
        yp = PREV ? a.yprev + (size_t)col * a.ldp : nullptr;
        out = a.out + (size_t)col * a.ldo;
        own = 2 * lp < a.ty;
        bufe = (a.ty + 2 * R) * PITCH;
        bool c1;
        pofs[0] = unit_ofs(y0 + 2 * lp, z0 + VZ * lz, own, cut);
        pofs[1] = unit_ofs(y0 + 2 * lp + 1, z0 + VZ * lz, own, c1);
        // lanes past the patch read (and discard) its first unit
        L0 = lds + (own ? (R + 2 * lp) * PITCH + PADZ + VZ * lz : R * PITCH + PADZ);
        const int yunits = 2 * R * a.lpr, nhalo = yunits + (a.zhalo ? a.ty * 2 * ZU : 0);
#pragma unroll
        for (int i = 0; i < NH; ++i) {
            const int e = tid + i * nt;
            int lrow = 0, gz = -1, lcol = 0;
            if (e < yunits) {
                const int hy = e / a.lpr, hu = e - hy * a.lpr;
                lrow = hy < R ? hy : hy + a.ty;
                gz = z0 + VZ * hu;
                lcol = PADZ + VZ * hu;
            } else if (e < nhalo) {
                const int r = (e - yunits) / (2 * ZU), hu = (e - yunits) % (2 * ZU);
                lrow = R + r;
                lcol = hu < ZU ? VZ * hu : PADZ + a.tz + VZ * (hu - ZU);
                gz = z0 - PADZ + lcol;
            }
            hofs[i] = unit_ofs(y0 - R + lrow, gz, e < nhalo, hcut[i]);
            // units off the grid stay at the zeros written below
            Lh[i] = hofs[i] != kOutside ? lds + lrow * PITCH + lcol : nullptr;
        }
        const V zero = {};
        for (int e = tid * VZ; e < 2 * bufe; e += nt * VZ) *(V *)&lds[e] = zero;

        const int xs = chunk * a.chunk_x, xe = min(a.n1, xs + a.chunk_x);
#pragma unroll
        for (int d = 0; d < 2 * R; ++d) {
            const auto rq = plane_rsrc(yk, xs - R + d, a.n1, P);
#pragma unroll
            for (int r = 0; r < 2; ++r) q[r][d] = place(vload<T, 0>(rq, pofs[r]), cut);
        }
        load_head(xs);
        load_point(xs);
        __syncthreads();
        int buf = 0;
        for (int x0 = xs; x0 < xe; x0 += QL) {
            run_block<0>(x0, xe, buf);
            buf = bufe - buf;  // an odd number of planes per block
        }
    }
};

}  // namespace sparc
