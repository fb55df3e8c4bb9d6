// Vector step: one pass over an orbital block computes, for every node x and
// column c,
//     out(x,c) = alpha * ( -1/2 lap_h yk + (V_eff(x) - shift) yk )(x,c) - beta * yprev(x,c)
// the local part of one step of the three-term Chebyshev recurrence of Sec.
// 3.4 (its first step without yprev, or a plain application of H), with the
// stencil of Sec. 3.1 Eq. FD:Laplacian and f = 0 off the grid.  The same
// launch gathers the projections chi_Jp^T yk of the input on the matrix cores
// (its last workgroups); the projector scatter that follows adds
// alpha V_nl yk (Sec. 3.1 Eq. non-localPS:FD).
//
// Data movement (HBM-bound):
//  * A workgroup owns a TY x TZ patch (TZ = 32, 64, 80 or 160 nodes) of the
//    (y, z) plane of one column and streams it along x (wider patches cut the
//    share of the z halo, whose two partial lines per row are fetched whole;
//    a patch as wide as the grid has none).  Each lane owns one unit of
//    consecutive z nodes of one y row: 4 FP32 or 2 FP64 values, 16 bytes, so
//    every global access is a 16-byte raw buffer load or store (a plain copy
//    with 4-byte accesses per lane reaches about 60% of the bandwidth of
//    16-byte accesses on this chip).  A lane keeps the 13 x-planes of its unit
//    in registers, one vector per plane (x neighbours never touch LDS); the
//    plane loop is unrolled over 26 planes so the queue rotates by register
//    renaming.
//  * The current plane of the patch plus its halo (6 rows in y; 8 FP32 / 6
//    FP64 nodes in z, whole units) is staged in LDS, double-buffered with one
//    barrier per plane; y and z neighbours are read there as 16-byte units.
//  * Loads are issued two planes ahead; points and planes outside the grid
//    fall outside the per-plane buffer descriptor's range (load zero, store
//    dropped).  The grid's z extent and every leading dimension must be
//    multiples of the unit, so a unit is either inside the grid or outside;
//    other grids take the row-pair kernel (rstep_kernel.hpp, which also takes
//    the larger FP32 blocks) or the scalar kernels (stencil.hip).
//  * Per point the sums run in the same order as in the scalar kernels.
//  * Workgroup indices are remapped so consecutive patches of one column run
//    on the same XCD and share halos in its L2 (optionally, col_group columns
//    of one patch run back to back and share V_eff); yprev and out are streamed
//    non-temporally when a step's blocks exceed the last-level cache.
//  * Orbital blocking (col_block = 2): one workgroup steps two columns of the
//    same patch, loading V_eff once for both and sharing the halo offsets and
//    the plane loop; each column keeps its own register queue and LDS plane.
#include <algorithm>
#include <cstring>
#include <type_traits>

#include "fstep_launch.hpp"
#include "rstep_launch.hpp"

namespace sparc {

static int vec_width(int dtype) { return dtype == SPARC_F64 ? 2 : 4; }

// patches offered per dtype (TY x TZ): FP64 8, 16, 32 x 32 and 8, 16, 24 x 64;
// FP32 16, 32, 64 x 32, 16, 32 x 64, 32 x 80 and 24 x 160 (128 to 960
// threads).  The wide ones cut the halo: a 24 x 160 patch spans a whole
// 160-node row, so it has no z halo at all and a y halo of 12 rows per 24.
static int vec_default_plan(int dtype) { return dtype == SPARC_F64 ? 1 : 2; }  // 16 x 32 FP64, 32 x 32 FP32

static int vec_nt(int dtype, int plan) { return (kPlanTZ[plan] / vec_width(dtype)) * kPlanTY[plan]; }

bool vec_plan_valid(int dtype, int plan)
{
    static const bool f64[kNumPlans] = {true, true, true, false, true, true, false, false, false, true};
    static const bool f32[kNumPlans] = {false, true, true, true, false, true, true, true, true, false};
    if (plan < 0 || plan >= kNumPlans) return false;
    return dtype == SPARC_F64 ? f64[plan] : f32[plan];
}

// two columns per workgroup double the register queues: only patches of at
// most 512 threads (whose waves may use 256 registers) take them
int vec_max_cblk(int dtype, int plan) { return vec_nt(dtype, plan) <= 512 ? 2 : 1; }

// split x so that about 8192 waves are in flight (at most kMaxChunks chunks,
// at least 4 planes each)
static int vec_default_chunks(const sparc_op *op, int dtype, int plan, int ns)
{
    const int ty = kPlanTY[plan], tz = kPlanTZ[plan];
    const long long tiles = (long long)((op->n[1] + ty - 1) / ty) * ((op->n[2] + tz - 1) / tz);
    const long long waves = tiles * ns * (vec_nt(dtype, plan) / 64);
    long long nch = (8192 + waves - 1) / waves;
    nch = std::max<long long>(1, std::min<long long>({nch, (long long)kMaxChunks, (long long)op->n[0] / 4}));
    return (int)nch;
}

bool vec_grid(const sparc_op *op, int dtype, std::initializer_list<int64_t> lds)
{
    const int vz = vec_width(dtype);
    if (op->n[2] % vz != 0) return false;
    for (int64_t ld : lds)
        if (ld % vz != 0) return false;
    return true;
}

static void set_chunks(const sparc_op *op, int nch, FLaunch &L)
{
    nch = std::max(1, std::min(nch, std::min(kMaxChunks, op->n[0])));
    L.chunk_x = (op->n[0] + nch - 1) / nch;
    L.nchunks = (op->n[0] + L.chunk_x - 1) / L.chunk_x;
}

// ---------------------------------------------------------------- row-pair launches


// LDS row pitch of a patch tz nodes wide: the narrowest of the two compiled
static int rstep_pitch(int dtype, int tz)
{
    const int need = tz + 2 * (dtype == SPARC_F64 ? 6 : 8);
    if (dtype == SPARC_F64) return need <= 44 ? 44 : need <= 108 ? 108 : 0;
    return need <= 112 ? 112 : need <= 176 ? 176 : 0;
}

// patch extent along z: whole rows or equal parts of them
static int rstep_tz(const sparc_op *op, int dtype)
{
    const int vz = vec_width(dtype), maxtz = dtype == SPARC_F64 ? 96 : 160;
    const int kz = (op->n[2] + maxtz - 1) / maxtz;
    return ((op->n[2] + kz - 1) / kz + vz - 1) / vz * vz;
}

// threads of a patch (whole waves; 0: the patch does not fit a workgroup)
static int rstep_threads(const sparc_op *op, int dtype, int tz, int ty, int &nh)
{
    const int vz = vec_width(dtype), lpr = tz / vz;
    const int pitch = rstep_pitch(dtype, tz);
    const int nt = (lpr * (ty / 2) + 63) / 64 * 64;
    if (!pitch || nt > kRThreads) return 0;
    if (2 * (size_t)(ty + 2 * kMaxRadius) * pitch * elem_size(dtype) > 65536) return 0;
    const int zu = dtype == SPARC_F64 ? 3 : 2;
    const int nhalo = 2 * kMaxRadius * lpr + (tz < op->n[2] ? ty * 2 * zu : 0);
    nh = (nhalo + nt - 1) / nt;
    return nh <= 2 ? nt : 0;
}

// Patch and x split of the row-pair kernels for ns columns (L.plan stays -1
// when no patch fits).  A workgroup holds its CU's SIMDs with up to 8 waves of
// 256 registers, so small launches run in a few rounds of workgroups and what
// decides is how full the last round is against the 12 planes every workgroup
// reads before its first output (worth about 10 planes).  The estimate is
//   (rounds + 1/2) x waves per CU x (planes + 10) x (1 + 4 / patch rows),
// the last factor the y halo.  Measured per step, FP32: 128^3 x 128 in 1, 2, 4
// x-chunks 733, 666, 688 us; 75 x 83 x 91 x 64 in 2, 4, 5 chunks 95, 101, 113
// us; 96^3 x 64 in 1, 4, 8 chunks 137, 138, 160 us.  Patches are as wide as the
// grid row where it fits (no z halo): 160^3 x 600 24 x 160 5.81 ms, 24 x 80
// 6.76 ms.  The estimate knows nothing of the L2: 160^3 x 600 in 4 x-chunks and
// groups of 4 columns takes 5.71 ms, its own choice (no x split, groups of 2)
// 5.85 ms; the autotuner finds the former.
// only_ty: the patch's rows, set by hand (0: chosen here).
static void choose_rstep(const sparc_op *op, int dtype, int ns, FLaunch &L, int only_ty = 0)
{
    if (op->n[2] < vec_width(dtype)) return;  // a cut row is read as its last whole unit
    const int tz = rstep_tz(op, dtype);
    const int tiles_z = (op->n[2] + tz - 1) / tz;
    // Workgroups of one patch of `group` columns run back to back and share its
    // V_eff in the XCD's L2.  Fields below 2 MB stay there by themselves (80 x 72
    // x 80 x 72 columns: 1.531 ms, by eight 1.554); from there eight columns pay
    // (96^3 x 64: 3.54 -> 3.24 ms, 128 x 120 x 128 x 14 by two 1.43 -> 1.30), above
    // 8 MB two (152 x 156 x 148 x 50: 8.36 -> 8.04; 160^3 x 600: 223.4 either
    // way, by eight 232.6, its halo rows leave the L2).  Only divisors of the
    // column count: a padded group would start workgroups for nothing (64 x 56 x
    // 72 x 100 by eight: 1.52 -> 1.75 ms).
    int group = 1;
    const int64_t field = op->nd * (int64_t)elem_size(dtype);
    for (int g = 2; field >= (int64_t)2 << 20 && g <= (field <= (int64_t)8 << 20 ? 8 : 2); g *= 2)
        if (ns % g == 0) group = g;
    double best = 0;
    for (int ky = 1; ky <= op->n[1]; ++ky) {
        const int ty = ((op->n[1] + ky - 1) / ky + 1) / 2 * 2;
        if (ty < 12 && ky > 1) break;
        if (only_ty > 0 && ty != only_ty) continue;
        int nh = 0;
        const int nt = rstep_threads(op, dtype, tz, ty, nh);
        // patches below 256 threads cannot host gather items (40 x 32 x 32 x
        // 503: 128 threads and a gather launch 57 us per step, 32 x 32 patches
        // of the other kernels 55 us)
        if (!nt || (nt < 256 && op->natoms > 0)) continue;
        const int w = nt / 64;
        // workgroups of about 10 planes: too few leave CUs idle (118 x 149 x 129
        // x 3: 177 of them, 40 us per step against the scalar kernels' 37.6 us)
        if (only_ty == 0 && (double)ns * ky * tiles_z * op->n[0] < 4000.0) continue;
        const size_t lds = 2 * (size_t)(ty + 2 * kMaxRadius) * rstep_pitch(dtype, tz) * elem_size(dtype);
        const int percu = std::max(1, std::min(8 / w, (int)(163840 / lds)));
        const int full = std::max(6, percu * w);  // fewer waves than that leave a CU waiting
        for (int nch = 1; nch <= kMaxChunks && (nch == 1 || op->n[0] / nch >= 8); ++nch) {
            const int cx = (op->n[0] + nch - 1) / nch, chunks = (op->n[0] + cx - 1) / cx;
            const long long wgs = (long long)ns * ((op->n[1] + ty - 1) / ty) * tiles_z * chunks;
            const long long slots = 256LL * percu, rem = wgs % slots;
            double rounds = (double)(wgs / slots) * full + 0.5 * full;
            if (rem) rounds += std::max<long long>(6, (rem + 255) / 256 * w);
            const double cost = rounds * (cx + 10) * (1.0 + 4.0 / ty);
            if (L.plan < 0 || cost < best) {
                best = cost;
                L.plan = kRowPair;
                L.tz = tz;
                L.ty = ty;
                L.chunk_x = cx;
                L.nchunks = chunks;
                L.cgroup = group;
                L.cblk = 1;
            }
        }
    }
}

// Whether the library's own choice is the row-pair kernels.  aligned: the
// 16-byte-unit kernels of this file take the grid too.
//  * FP32 from 4e6 values per block: 160^3 x 600 7.75 -> 6.84 ms per step
//    launch with the projections in its tail (without, as it runs beside
//    gather_whole_kernel, 5.85 ms), 128^3 x 128 827 -> 666 us, 96^3 x 64 178 ->
//    137 us, 64^3 x 64 49 -> 44 us; below (32^3 x 64) 12 -> 15 us.
//  * FP64, whose step is bound by memory already: only where the 16 x 32 patches
//    of the other kernels reach 15 % past the grid (75 x 83 x 92 x 37 151 -> 131
//    us; 96^3 x 64, no overhang, 300 -> 322 us).
//  * Rows of broken units, which only the scalar kernels take otherwise:
//    75 x 83 x 91, FP64 x 37 171 -> 135 us, FP32 x 64 191 -> 95 us.
static bool take_rstep(const sparc_op *op, int dtype, int ns, bool aligned)
{
    if ((double)op->nd * ns < 4e6 || op->n[2] < vec_width(dtype)) return false;
    if (!aligned || dtype == SPARC_F32) return true;
    const double pad = (double)((op->n[1] + 15) / 16 * 16) * ((op->n[2] + 31) / 32 * 32);
    return pad >= 1.15 * op->n[1] * op->n[2];
}

bool rstep_patch(const sparc_op *op, int dtype, int tz, int ty)
{
    FLaunch L;
    if (tz == rstep_tz(op, dtype) && ty > 0) choose_rstep(op, dtype, 1, L, ty);
    return L.plan >= 0;
}

FLaunch choose_vec_launch(const sparc_op *op, int dtype, int ns, std::initializer_list<int64_t> lds)
{
    FLaunch L;
    const bool aligned = vec_grid(op, dtype, lds);
    const bool tuned = tune_applies(op, dtype, ns);
    // a patch set by hand that both kinds of kernels offer goes to the one the
    // library takes for the block itself
    const int ty = op->tune_ty[dtype];
    const bool both = ty > 0 && op->tune_shape[dtype] >= 0 && op->tune_shape[dtype] != kRowPair &&
                      op->tune_cblk[dtype] != 2 && take_rstep(op, dtype, ns, aligned) &&
                      rstep_patch(op, dtype, kPlanTZ[op->tune_shape[dtype]], ty);
    if (tuned && (op->tune_shape[dtype] == kRowPair || both)) {
        choose_rstep(op, dtype, ns, L, ty);
        if (L.plan >= 0 && op->tune_chunk[dtype] > 0) set_chunks(op, (op->n[0] + op->tune_chunk[dtype] - 1) / op->tune_chunk[dtype], L);
        if (L.plan >= 0 && op->tune_group[dtype] > 0) L.cgroup = op->tune_group[dtype];
        if (L.plan >= 0) return L;
    }
    const bool forced = tuned && (op->tune_shape[dtype] >= 0 || op->tune_chunk[dtype] > 0 || op->tune_group[dtype] > 0 ||
                                  op->tune_cblk[dtype] > 0);
    if (!(aligned && forced) && take_rstep(op, dtype, ns, aligned)) choose_rstep(op, dtype, ns, L);
    if (L.plan >= 0 || !aligned) return L;
    int plan = vec_default_plan(dtype);
    if (tuned && op->tune_shape[dtype] >= 0 && vec_plan_valid(dtype, op->tune_shape[dtype]))
        plan = op->tune_shape[dtype];
    int nch = vec_default_chunks(op, dtype, plan, ns);
    if (tuned && op->tune_chunk[dtype] > 0) nch = (op->n[0] + op->tune_chunk[dtype] - 1) / op->tune_chunk[dtype];
    L.plan = plan;
    set_chunks(op, nch, L);
    L.cgroup = (tuned && op->tune_group[dtype] > 0) ? op->tune_group[dtype] : 1;
    L.cblk = (tuned && op->tune_cblk[dtype] == 2 && vec_max_cblk(dtype, plan) == 2) ? 2 : 1;
    return L;
}

FLaunch vec_launch_plan(const sparc_op *op, int dtype, int ns, int plan)
{
    FLaunch L;
    L.plan = plan;
    set_chunks(op, vec_default_chunks(op, dtype, plan, ns), L);
    return L;
}

template <typename T>
static int launch_rstep_t(const sparc_op *op, const FLaunch &L, const void *yk, int64_t ldk, const void *yprev,
                          int64_t ldp, void *out, int64_t ldo, int ns, void *part, const StepCoef &c,
                          hipStream_t stream)
{
    constexpr int dtype = std::is_same<T, double>::value ? SPARC_F64 : SPARC_F32;
    int nh = 0;
    const int nt = rstep_threads(op, dtype, L.tz, L.ty, nh);
    if (!nt) return fail(SPARC_E_ARG, "row-pair patch does not fit a workgroup");
    RStepArgs<T> a;
    std::memset(&a, 0, sizeof(a));
    a.yk = (const T *)yk;
    a.yprev = (const T *)yprev;
    a.out = (T *)out;
    a.veff = std::is_same<T, double>::value ? (const T *)op->d_veff64 : (const T *)op->d_veff32;
    a.ldk = ldk;
    a.ldp = ldp;
    a.ldo = ldo;
    a.n1 = op->n[0];
    a.n2 = op->n[1];
    a.n3 = op->n[2];
    a.tz = L.tz;
    a.ty = L.ty;
    a.lpr = L.tz / VecTraits<T>::N;
    a.tiles_y = (op->n[1] + L.ty - 1) / L.ty;
    a.tiles_z = (op->n[2] + L.tz - 1) / L.tz;
    a.zhalo = L.tz < op->n[2] ? 1 : 0;
    a.chunk_x = L.chunk_x;
    a.nchunks = L.nchunks;
    const int G = std::max(1, std::min(L.cgroup, ns));
    const long long nb = (long long)(ns + G - 1) / G * G * L.nchunks * a.tiles_y * a.tiles_z;
    if (nb > 0x7fffffffLL) return fail(SPARC_E_SHAPE, "too many workgroups for one launch");
    a.nblocks = (int)nb;
    a.ns = ns;
    a.cgroup = G;
    a.c0 = (T)(-3.0 * op->w[0]);
    for (int p = 1; p <= kMaxRadius; ++p) a.cp[p - 1] = (T)(-0.5 * op->w[p]);
    a.alpha = (T)c.alpha;
    a.beta = (T)c.beta;
    a.shift = (T)c.shift;
    const bool prev = c.has_prev && yprev != nullptr;
    const bool strm = (double)op->nd * ns * 3 * sizeof(T) > kStreamBytes;
    GatherArgs<T, T> g;
    std::memset(&g, 0, sizeof(g));
    int ncb = 0, nitems = 0, ngb = 0;
    if (part && op->natoms > 0) {
        if ((long long)(ns + 15) / 16 > 65535) return fail(SPARC_E_SHAPE, "too many columns for one gather launch");
        if (nt < 256) return fail(SPARC_E_ARG, "row-pair patch too small to gather projections");
        g.Y = (const T *)yk;
        g.ldy = ldk;
        g.ns = ns;
        g.nproj_total = op->nproj_total;
        g.atoms = op->d_atoms;
        g.small = op->nd < kUnit;
        g.units = (const int2 *)op->d_units;
        g.chiu = std::is_same<T, double>::value ? (const T *)op->d_chiu64 : (const T *)op->d_chiu32;
        g.box_off = op->d_box_off;
        g.chi = std::is_same<T, double>::value ? (const T *)op->d_chi64 : (const T *)op->d_chi32;
        g.part = (T *)part;
        ncb = (ns + 15) / 16;
        nitems = op->natoms * ncb * kGatherSplit;
        const int per = nt / 256;
        ngb = (nitems + per - 1) / per;
        if ((long long)a.nblocks + ngb > 0x7fffffffLL) return fail(SPARC_E_SHAPE, "too many workgroups for one launch");
    }
    ProfScope prof(prev ? 0 : 3, stream);
    const int natoms = std::max(op->natoms, 1);
    const int rag = (VecTraits<T>::N - op->n[2] % VecTraits<T>::N) % VecTraits<T>::N;
    const bool wide = rstep_pitch(dtype, L.tz) == (dtype == SPARC_F64 ? 108 : 176);
#define SPARC_RSTEP(name) name(a, g, natoms, ncb, nitems, ngb, nt, nh, prev, strm, stream)
    if constexpr (std::is_same<T, float>::value) {
        switch (rag) {
            case 0: return wide ? SPARC_RSTEP(rstep_f32_p176) : SPARC_RSTEP(rstep_f32_p112);
            case 1: return wide ? SPARC_RSTEP(rstep_f32_p176_r1) : SPARC_RSTEP(rstep_f32_p112_r1);
            case 2: return wide ? SPARC_RSTEP(rstep_f32_p176_r2) : SPARC_RSTEP(rstep_f32_p112_r2);
            default: return wide ? SPARC_RSTEP(rstep_f32_p176_r3) : SPARC_RSTEP(rstep_f32_p112_r3);
        }
    } else {
        if (rag) return wide ? SPARC_RSTEP(rstep_f64_p108_r1) : SPARC_RSTEP(rstep_f64_p44_r1);
        return wide ? SPARC_RSTEP(rstep_f64_p108) : SPARC_RSTEP(rstep_f64_p44);
    }
#undef SPARC_RSTEP
}

template <typename T>
static int launch_fstep_t(const sparc_op *op, const FLaunch &L, const void *yk, int64_t ldk, const void *yprev,
                          int64_t ldp, void *out, int64_t ldo, int ns, void *part, const StepCoef &c,
                          hipStream_t stream)
{
    const int ty = kPlanTY[L.plan], tz = kPlanTZ[L.plan];
    const int nt = (tz / VecTraits<T>::N) * ty;
    FStepArgs<T> a;
    std::memset(&a, 0, sizeof(a));
    a.yk = (const T *)yk;
    a.yprev = (const T *)yprev;
    a.out = (T *)out;
    a.veff = std::is_same<T, double>::value ? (const T *)op->d_veff64 : (const T *)op->d_veff32;
    a.ldk = ldk;
    a.ldp = ldp;
    a.ldo = ldo;
    a.n1 = op->n[0];
    a.n2 = op->n[1];
    a.n3 = op->n[2];
    a.tiles_y = (op->n[1] + ty - 1) / ty;
    a.tiles_z = (op->n[2] + tz - 1) / tz;
    a.chunk_x = L.chunk_x;
    a.nchunks = L.nchunks;
    const int cb = L.cblk == 2 ? 2 : 1;
    const int ngroups = (ns + cb - 1) / cb;  // column blocks
    const int G = std::max(1, std::min(L.cgroup, ngroups));
    const long long nb = (long long)(ngroups + G - 1) / G * G * L.nchunks * a.tiles_y * a.tiles_z;
    if (nb > 0x7fffffffLL) return fail(SPARC_E_SHAPE, "too many workgroups for one launch");
    a.nblocks = (int)nb;
    a.remap = 1;
    a.ns = ns;
    a.cgroup = G;
    a.c0 = (T)(-3.0 * op->w[0]);
    for (int p = 1; p <= kMaxRadius; ++p) a.cp[p - 1] = (T)(-0.5 * op->w[p]);
    a.alpha = (T)c.alpha;
    a.beta = (T)c.beta;
    a.shift = (T)c.shift;
    const bool prev = c.has_prev && yprev != nullptr;
    // blocks the last-level cache cannot keep between steps are streamed
    const bool strm = (double)op->nd * ns * 3 * sizeof(T) > kStreamBytes;
    GatherArgs<T, T> g;
    std::memset(&g, 0, sizeof(g));
    int ncb = 0, nitems = 0, ngb = 0;
    if (part && op->natoms > 0) {
        if ((long long)(ns + 15) / 16 > 65535) return fail(SPARC_E_SHAPE, "too many columns for one gather launch");
        if (nt < 256) {
            // the patch is too small to host gather items: a launch of its own
            int st;
            if ((st = launch_gather(op, std::is_same<T, double>::value ? SPARC_F64 : SPARC_F32, yk, ldk, ns, part,
                                    kGatherSplit, stream)))
                return st;
        } else {
            g.Y = (const T *)yk;
            g.ldy = ldk;
            g.ns = ns;
            g.nproj_total = op->nproj_total;
            g.atoms = op->d_atoms;
            g.small = op->nd < kUnit;
            g.units = (const int2 *)op->d_units;
            g.chiu = std::is_same<T, double>::value ? (const T *)op->d_chiu64 : (const T *)op->d_chiu32;
            g.box_off = op->d_box_off;
            g.chi = std::is_same<T, double>::value ? (const T *)op->d_chi64 : (const T *)op->d_chi32;
            g.part = (T *)part;
            ncb = (ns + 15) / 16;
            nitems = op->natoms * ncb * kGatherSplit;
            const int per = nt / 256;
            ngb = (nitems + per - 1) / per;
            if ((long long)a.nblocks + ngb > 0x7fffffffLL) return fail(SPARC_E_SHAPE, "too many workgroups for one launch");
        }
    }
    ProfScope prof(prev ? 0 : 3, stream);
    const int natoms = std::max(op->natoms, 1);
    if constexpr (std::is_same<T, float>::value) {
        if (tz == 160) {
            if (ty == 24) return fstep_f32_ty24_tz160(a, g, natoms, ncb, nitems, ngb, prev, strm, cb, stream);
        } else if (tz == 80) {
            if (ty == 32) return fstep_f32_ty32_tz80(a, g, natoms, ncb, nitems, ngb, prev, strm, cb, stream);
        } else if (tz == 64) {
            switch (ty) {
                case 16: return fstep_f32_ty16_tz64(a, g, natoms, ncb, nitems, ngb, prev, strm, cb, stream);
                case 32: return fstep_f32_ty32_tz64(a, g, natoms, ncb, nitems, ngb, prev, strm, cb, stream);
            }
        } else {
            switch (ty) {
                case 16: return fstep_f32_ty16(a, g, natoms, ncb, nitems, ngb, prev, strm, cb, stream);
                case 32: return fstep_f32_ty32(a, g, natoms, ncb, nitems, ngb, prev, strm, cb, stream);
                case 64: return fstep_f32_ty64(a, g, natoms, ncb, nitems, ngb, prev, strm, cb, stream);
            }
        }
    } else {
        if (tz == 64) {
            switch (ty) {
                case 8: return fstep_f64_ty8_tz64(a, g, natoms, ncb, nitems, ngb, prev, strm, cb, stream);
                case 16: return fstep_f64_ty16_tz64(a, g, natoms, ncb, nitems, ngb, prev, strm, cb, stream);
                case 24: return fstep_f64_ty24_tz64(a, g, natoms, ncb, nitems, ngb, prev, strm, cb, stream);
            }
        } else {
            switch (ty) {
                case 8: return fstep_f64_ty8(a, g, natoms, ncb, nitems, ngb, prev, strm, cb, stream);
                case 16: return fstep_f64_ty16(a, g, natoms, ncb, nitems, ngb, prev, strm, cb, stream);
                case 32: return fstep_f64_ty32(a, g, natoms, ncb, nitems, ngb, prev, strm, cb, stream);
            }
        }
    }
    return fail(SPARC_E_ARG, "patch height not available for this dtype");
}

int launch_fstep(const sparc_op *op, int dtype, const FLaunch &L, const void *yk, int64_t ldk, const void *yprev,
                 int64_t ldp, void *out, int64_t ldo, int ns, void *part, const StepCoef &c, hipStream_t stream)
{
    if (L.plan < 0) return fail(SPARC_E_ARG, "vector step not available");
    if (L.plan == kRowPair) {
        if (dtype == SPARC_F64)
            return launch_rstep_t<double>(op, L, yk, ldk, yprev, ldp, out, ldo, ns, part, c, stream);
        return launch_rstep_t<float>(op, L, yk, ldk, yprev, ldp, out, ldo, ns, part, c, stream);
    }
    if (dtype == SPARC_F64)
        return launch_fstep_t<double>(op, L, yk, ldk, yprev, ldp, out, ldo, ns, part, c, stream);
    return launch_fstep_t<float>(op, L, yk, ldk, yprev, ldp, out, ldo, ns, part, c, stream);
}

}  // namespace sparc
