// Nonlocal pseudopotential term of H (Sec. 2 Eq. V_nl; Sec. 3.1 Eq.
// non-localPS:FD):  (V_nl y)(x) = sum_J sum_p chi_Jp(x) * h^3 gamma_Jp * (chi_Jp^T y).
//
// Two kernels:
//  * gather: per atom J, the projections S_Jp(c) = sum_{x in cube_J} chi_Jp(x) y(x,c)
//    as a small dense GEMM on the matrix cores, S_J^T (ns x nproj) =
//    Y_cube^T (ns x nbox) * chi_J (nbox x nproj), using
//    v_mfma_f64_16x16x4f64 (FP64) or v_mfma_f32_16x16x4f32 (FP32).  The cube is
//    read (for FP32 blocks) as units of 4 nodes along z, 16 bytes per lane, four
//    matrix instructions per load; the units (the K dimension) are cut into 4
//    kGatherSplit segments of one wave each.  Either kGatherSplit workgroups
//    share an atom and 16 columns and leave partial 16 x nproj tiles that the
//    consumer sums in split order, or one workgroup sums them itself in the
//    same order; no atomics, the same bits either way.
//    What bounds it: the cube rows are short (14 to 15 nodes), so each costs
//    1.5 lines of 128 bytes per column, 3.3 GB at 160^3 x 600 with 128 cubes.
//    Node by node (4 bytes per lane, a table entry and a chi value per matrix
//    instruction) the gather took 948 us there, by units of 4 nodes 676 us
//    (4.9 TB/s of those lines).
//  * scatter: out(x,c) += alpha * sum_{J: x in cube_J} sum_p chi_Jp(x) h^3 gamma_Jp S_Jp(c)
//    over the unique nodes covered by at least one cube, grouped in blocks of
//    at most 256 nodes that touch at most kScatterSlots atoms (tables built at
//    operator creation).  A workgroup first requests its nodes' out values for
//    32 FP32 / 8 FP64 columns (8 when the block tables are too large for
//    LDS), finishes h^3 gamma S for its block's atoms and those columns into
//    LDS (split partials summed in order), then each thread updates one node
//    for all of them, atoms in a fixed order: deterministic even where cubes
//    overlap.  The cube rows are short (a few tens of bytes per column), so
//    the kernel's HBM traffic is set by partial lines and its time by the
//    scattered read-modify-write of out, not by the table or chi reads.
//
// MFMA operand layout of the 16x16x4 instructions (64 lanes, lane = i + 16k,
// i in 0..15, k in 0..3): lane supplies A[i][k] (column c0+i at cube point
// k of the current group of 4) and B[k][j] (projector j at that point).  The
// FP32 accumulator keeps D[4*(lane/16) + r][lane%16] in register r; the FP64
// accumulator keeps D[lane/16 + 4*r][lane%16].
#include <algorithm>

#include "nonlocal_kernel.hpp"

namespace sparc {

template <typename T, typename TI>
__global__ void __launch_bounds__(256) gather_kernel(const GatherArgs<T, TI> g)
{
    __shared__ T tile[4][16][16];
    gather_item<T, TI>(g, blockIdx.x, blockIdx.y, blockIdx.z, tile, threadIdx.x);
}

template <typename T, typename TI>
__global__ void __launch_bounds__(256) gather_whole_kernel(const GatherArgs<T, TI> g)
{
    __shared__ T tile[4][4][16][16];
    gather_whole<T, TI>(g, blockIdx.y, blockIdx.x, tile);
}

// table in dynamic LDS: [block's atoms][npm][NC]
template <typename T, int NC, int NP>
__global__ void __launch_bounds__(256) scatter_kernel(const ScatterArgs<T> s, int npm)
{
    extern __shared__ __align__(16) char scatter_lds[];
    scatter_item<T, NC, NP>(s, blockIdx.x, blockIdx.y, (T *)scatter_lds, npm);
}

// blockIdx.x: atom.  chi at the places append_units gives the cube's nodes, and
// chi in FP32.
__global__ void __launch_bounds__(256) unit_chi_kernel(const AtomDev *atoms, const double *chi, float *chi32, int n2,
                                                       int n3, long long nd, double *chiu64, float *chiu32)
{
    const AtomDev A = atoms[blockIdx.x];
    const int nbox = A.ext[0] * A.ext[1] * A.ext[2];
    const int s0 = A.lo[2] / kUnit, per_row = (A.lo[2] + A.ext[2] - 1) / kUnit - s0 + 1;
    for (int t = blockIdx.y * 256 + threadIdx.x; t < nbox; t += gridDim.y * 256) {
        const int r = t / A.ext[2], z = A.lo[2] + t % A.ext[2], s = z / kUnit;
        const long long row = (long long)n3 * ((A.lo[1] + r % A.ext[1]) + (long long)n2 * (A.lo[0] + r / A.ext[1]));
        const long long first = max(0LL, min(row + kUnit * s, nd - kUnit));
        const int d = kUnit * (r * per_row + s - s0) + (int)(row + z - first);
        for (int p = 0; p < A.nproj; ++p) {
            const double v = chi[A.chi0 + (long long)p * nbox + t];
            const long long o = A.chiu0 + (long long)p * A.nunits * kUnit + d;
            chi32[A.chi0 + (long long)p * nbox + t] = (float)v;
            chiu64[o] = v;
            chiu32[o] = (float)v;
        }
    }
}

int build_unit_chi(sparc_op *op, int64_t total)
{
    hipError_t e = hipMemset(op->d_chiu64, 0, total * sizeof(double));
    if (e == hipSuccess) e = hipMemset(op->d_chiu32, 0, total * sizeof(float));
    if (e == hipSuccess) {
        hipLaunchKernelGGL(unit_chi_kernel, dim3(op->natoms, 4), dim3(256), 0, 0, op->d_atoms, op->d_chi64,
                           op->d_chi32, op->n[1], op->n[2], op->nd, op->d_chiu64, op->d_chiu32);
        e = hipGetLastError();
    }
    return e == hipSuccess ? SPARC_OK : fail(SPARC_E_HIP, std::string("projector tables: ") + hipGetErrorString(e));
}

bool gather_wide(const sparc_op *op, int ns)
{
    // FP32 filters, per step with a workgroup per pair against the step's tail:
    // 64 pairs (96^3, 16 atoms x 64 columns) 168 and 148 us, 400 (40^3, 40 x 160)
    // 99 and 94, 512 (64^3, 32 x 256) 239 and 237; 1024 (128^3, 64 x 256) 1402 and
    // 1459, 1178 (120^3, 31 x 600) 2770 and 2862, 2048 (160^3, 128 x 256) 3127 and
    // 3377, 4864 (160^3, 128 x 600) 7182 and 7306
    return (long long)op->natoms * ((ns + 15) / 16) >= 1024;
}

template <typename T, typename TI = T>
static int launch_gather_t(const sparc_op *op, const void *Y, int64_t ldy, int ns, void *part, int nparts,
                           hipStream_t stream, const T *chi, const T *chiu)
{
    GatherArgs<T, TI> a;
    a.Y = (const TI *)Y;
    a.ldy = ldy;
    a.ns = ns;
    a.nproj_total = op->nproj_total;
    a.small = op->nd < kUnit;
    a.atoms = op->d_atoms;
    a.units = (const int2 *)op->d_units;
    a.chiu = chiu;
    a.box_off = op->d_box_off;
    a.chi = chi;
    a.part = (T *)part;
    const unsigned ncb = (unsigned)(ns + 15) / 16;
    ProfScope prof(1, stream);
    if constexpr (sizeof(TI) == 4) {
        if (nparts == 1) {
            for (int J = 0; J < op->natoms; J += 65535) {  // rows of a grid
                a.atoms = op->d_atoms + J;
                hipLaunchKernelGGL((gather_whole_kernel<T, TI>), dim3(ncb, std::min(op->natoms - J, 65535)), dim3(256), 0,
                                   stream, a);
            }
            SPARC_HIP(hipGetLastError());
            return SPARC_OK;
        }
    }
    hipLaunchKernelGGL((gather_kernel<T, TI>), dim3(op->natoms, ncb, kGatherSplit), dim3(256), 0, stream, a);
    SPARC_HIP(hipGetLastError());
    return SPARC_OK;
}

int launch_gather_f32_to_f64(const sparc_op *op, const float *Y, int64_t ldy, int ns, double *part, int nparts,
                             hipStream_t stream)
{
    if (op->natoms == 0) return SPARC_OK;
    if ((long long)(ns + 15) / 16 > 65535) return fail(SPARC_E_SHAPE, "too many columns for one gather launch");
    return launch_gather_t<double, float>(op, Y, ldy, ns, part, nparts, stream, op->d_chi64, op->d_chiu64);
}

int launch_gather(const sparc_op *op, int dtype, const void *Y, int64_t ldy, int ns, void *part, int nparts,
                  hipStream_t stream)
{
    if (op->natoms == 0) return SPARC_OK;
    if ((long long)(ns + 15) / 16 > 65535) return fail(SPARC_E_SHAPE, "too many columns for one gather launch");
    if (dtype == SPARC_F64) return launch_gather_t<double>(op, Y, ldy, ns, part, nparts, stream, op->d_chi64, op->d_chiu64);
    return launch_gather_t<float>(op, Y, ldy, ns, part, nparts, stream, op->d_chi32, op->d_chiu32);
}

template <typename T>
static int launch_scatter_t(const sparc_op *op, void *out, int64_t ldo, int ns, const void *part, int nparts, double alpha,
                            hipStream_t stream, const T *chi, const T *chiu, const T *hg)
{
    ScatterArgs<T> a;
    a.out = (T *)out;
    a.ldo = ldo;
    a.ns = ns;
    a.nproj_total = op->nproj_total;
    a.blk_pt = op->d_nl_blk_pt;
    a.blk_at = op->d_nl_blk_at;
    a.blk_atoms = op->d_nl_blk_atoms;
    a.pts = op->d_nl_pts;
    a.ent_off = op->d_nl_off;
    // FP32 blocks read chi in the unit layout, which their gather has just
    // brought into the caches (32^3 x 106: 9.95 us from its own copy)
    const bool units = sizeof(T) == 4 && op->d_nl_entu;
    a.ent = (const int4 *)(units ? op->d_nl_entu : op->d_nl_ent);
    a.atoms = op->d_atoms;
    a.chi = units ? chiu : chi;
    a.hg = hg;
    a.part = (const T *)part;
    a.alpha = (T)alpha;
    // columns per workgroup: FP32 blocks take 32 when the table fits in 32
    // KiB of LDS (a quarter of the chi and table reads of 8 columns, same
    // time); FP64 blocks keep 8 (16 measured slower)
    constexpr int NW = sizeof(T) == 4 ? 32 : kScatterCols;
    const int npm = std::max(1, op->max_nproj);
    const size_t row = (size_t)std::max(1, op->nl_max_slots) * npm * sizeof(T);
    const bool wide = row * NW <= 32768;
    const int nc = wide ? NW : kScatterCols;
    if ((ns + nc - 1) / nc > 65535) return fail(SPARC_E_SHAPE, "too many columns for one scatter launch");
    dim3 grid(op->nl_nblk, (ns + nc - 1) / nc);
    ProfScope prof(2, stream);
    const size_t lds = row * nc;
    if constexpr (NW != kScatterCols) {
        if (wide && nparts == 1)
            hipLaunchKernelGGL((scatter_kernel<T, NW, 1>), grid, dim3(256), lds, stream, a, npm);
        else if (wide)
            hipLaunchKernelGGL((scatter_kernel<T, NW, kGatherSplit>), grid, dim3(256), lds, stream, a, npm);
    }
    if (NW == kScatterCols || !wide) {
        if (nparts == 1)
            hipLaunchKernelGGL((scatter_kernel<T, kScatterCols, 1>), grid, dim3(256), lds, stream, a, npm);
        else
            hipLaunchKernelGGL((scatter_kernel<T, kScatterCols, kGatherSplit>), grid, dim3(256), lds, stream, a, npm);
    }
    SPARC_HIP(hipGetLastError());
    return SPARC_OK;
}

int launch_scatter(const sparc_op *op, int dtype, void *out, int64_t ldo, int ns, const void *part, int nparts,
                   double alpha, hipStream_t stream)
{
    if (op->natoms == 0) return SPARC_OK;
    if (dtype == SPARC_F64) return launch_scatter_t<double>(op, out, ldo, ns, part, nparts, alpha, stream, op->d_chi64, op->d_chiu64,
                                                            op->d_hg64);
    return launch_scatter_t<float>(op, out, ldo, ns, part, nparts, alpha, stream, op->d_chi32, op->d_chiu32, op->d_hg32);
}

}  // namespace sparc
