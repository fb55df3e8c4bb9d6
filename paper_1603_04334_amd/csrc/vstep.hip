// The step of one FP64 vector without Y_{k-1}: H v for Lanczos (with the
// projections of v gathered by the first workgroups of the launch) and A p for
// the Poisson solver (no potential), each with the partial sums of v.(out) per
// workgroup that the caller's next kernel finishes in a fixed order.
//
// One vector is small (7 MB at 96^3, 33 MB at 160^3) and stays in the caches;
// what costs time is getting enough workgroups in flight with few repeated
// planes.  16-byte units on patches of 16 x 32 nodes (256 threads), x cut so
// that about four workgroups share a CU: at 160^3 91.7 us per CG iteration
// (8 x 32: 93.9, 8 x 64: 93.6, 16 x 64: 93.8, 4 x 32: 96.0; 512 or 2048
// workgroups: 95.2, 93.4).
#include <algorithm>
#include <cstring>

#include "fstep_kernel.hpp"
#include "nonlocal_kernel.hpp"

namespace sparc {

constexpr int kVTY = 16, kVTZ = 32, kVThreads = kVTY * kVTZ / 2;

// fixed-order workgroup sum of the lanes' products
__device__ __forceinline__ void store_partial(double v, double *dot, int b)
{
    __shared__ double red[kVThreads / 64];
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = red[0];
        for (int i = 1; i < kVThreads / 64; ++i) t += red[i];
        dot[b] = t;
    }
}

// H u for Lanczos: the first ngather workgroups gather the projections of u
// (atom i % natoms, split i / natoms, as the standalone gather; ngather is a
// multiple of 8, so the step's XCD-aware index remap still sees the hardware
// round-robin), the rest step
template <int RAG>
__global__ void __launch_bounds__(kVThreads)
    vstep_gather_kernel(const FStepArgs<double> a, const GatherArgs<double, double> g, int natoms, int ngather,
                        double *dot)
{
    using K = FStep<double, kVTY, false, false, 1, kVTZ, true, true, RAG>;
    __shared__ __align__(16) union {
        typename K::Shared step;
        double tile[4][16][16];
    } sh;
    static_assert(kVThreads == 256, "one gather item per workgroup");
    if ((int)blockIdx.x < ngather) {
        gather_item<double, double>(g, blockIdx.x % natoms, 0, blockIdx.x / natoms, sh.tile, threadIdx.x);
        return;
    }
    const int b = blockIdx.x - ngather;
    K k(a);
    k.run(b, sh.step);
    store_partial(k.dacc, dot, b);
}

// A p without a potential; skipped when *done < iter
template <int RAG>
__global__ void __launch_bounds__(kVThreads)
    vstep_kernel(const FStepArgs<double> a, double *dot, const int *done, int iter)
{
    using K = FStep<double, kVTY, false, false, 1, kVTZ, false, true, RAG>;
    __shared__ __align__(16) typename K::Shared sh;
    if (*done < iter) return;
    K k(a);
    k.run(blockIdx.x, sh);
    store_partial(k.dacc, dot, blockIdx.x);
}

struct VPlan {
    int tiles_y, tiles_z, chunk_x, nchunks;
    long long blocks() const { return (long long)tiles_y * tiles_z * nchunks; }
};

static VPlan vstep_plan(const sparc_op *op)
{
    VPlan v;
    v.tiles_y = (op->n[1] + kVTY - 1) / kVTY;
    v.tiles_z = (op->n[2] + kVTZ - 1) / kVTZ;
    const long long want = 1024;  // workgroups: four to a CU
    const long long tiles = (long long)v.tiles_y * v.tiles_z;
    const long long nch = std::max<long long>(1, std::min<long long>((want + tiles - 1) / tiles, op->n[0] / 4));
    v.chunk_x = (int)((op->n[0] + nch - 1) / nch);
    v.nchunks = (op->n[0] + v.chunk_x - 1) / v.chunk_x;
    return v;
}

bool vstep_takes(const sparc_op *op) { return op->n[2] >= 2 && vstep_plan(op).blocks() <= 65536; }

long long vstep_blocks(const sparc_op *op) { return vstep_plan(op).blocks(); }

static FStepArgs<double> vstep_args(const sparc_op *op, const double *v, double *out, double alpha)
{
    const VPlan p = vstep_plan(op);
    FStepArgs<double> a;
    std::memset(&a, 0, sizeof(a));
    a.yk = v;
    a.out = out;
    a.veff = op->d_veff64;
    a.ldk = a.ldo = op->nd;
    a.n1 = op->n[0];
    a.n2 = op->n[1];
    a.n3 = op->n[2];
    a.tiles_y = p.tiles_y;
    a.tiles_z = p.tiles_z;
    a.nchunks = p.nchunks;
    a.chunk_x = p.chunk_x;
    a.nblocks = (int)p.blocks();
    a.remap = 1;
    a.ns = a.cgroup = 1;
    a.c0 = -3.0 * op->w[0];
    for (int q = 1; q <= kMaxRadius; ++q) a.cp[q - 1] = -0.5 * op->w[q];
    a.alpha = alpha;
    return a;
}

int launch_vstep_gather(const sparc_op *op, const double *v, double *out, double *dot, double *part, hipStream_t stream)
{
    const FStepArgs<double> a = vstep_args(op, v, out, 1.0);
    GatherArgs<double, double> g;
    std::memset(&g, 0, sizeof(g));
    g.Y = v;
    g.ldy = op->nd;
    g.ns = 1;
    g.nproj_total = op->nproj_total;
    g.small = op->nd < kUnit;
    g.atoms = op->d_atoms;
    g.box_off = op->d_box_off;
    g.chi = op->d_chi64;
    g.part = part;
    const int ngather = op->natoms * kGatherSplit;
    const dim3 grid((unsigned)(ngather + a.nblocks)), blk(kVThreads);
    ProfScope prof(3, stream);
    if (op->n[2] & 1)
        hipLaunchKernelGGL(vstep_gather_kernel<1>, grid, blk, 0, stream, a, g, std::max(1, op->natoms), ngather, dot);
    else
        hipLaunchKernelGGL(vstep_gather_kernel<0>, grid, blk, 0, stream, a, g, std::max(1, op->natoms), ngather, dot);
    SPARC_HIP(hipGetLastError());
    return SPARC_OK;
}

int launch_vstep(const sparc_op *op, const double *v, double *out, double alpha, double *dot, const int *done, int iter,
                 hipStream_t stream)
{
    const FStepArgs<double> a = vstep_args(op, v, out, alpha);
    const dim3 grid((unsigned)a.nblocks), blk(kVThreads);
    if (op->n[2] & 1)
        hipLaunchKernelGGL(vstep_kernel<1>, grid, blk, 0, stream, a, dot, done, iter);
    else
        hipLaunchKernelGGL(vstep_kernel<0>, grid, blk, 0, stream, a, dot, done, iter);
    SPARC_HIP(hipGetLastError());
    return SPARC_OK;
}

}  // namespace sparc
