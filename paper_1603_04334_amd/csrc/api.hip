// C ABI of the Chebyshev-filter library: operator construction, H application,
// the filter driver, status strings and per-kernel event timing.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <initializer_list>
#include <memory>
#include <new>

#include <rocprofiler-sdk-roctx/roctx.h>

#include "internal.hpp"

namespace sparc {

static thread_local std::string g_last_error;

void set_error(const std::string &msg) { g_last_error = msg; }

int fail(int status, const std::string &msg)
{
    set_error(msg);
    return status;
}

size_t elem_size(int dtype) { return dtype == SPARC_F64 ? sizeof(double) : sizeof(float); }

// ---------------------------------------------------------------- profiling

namespace {
struct ProfRec {
    int kernel;
    hipEvent_t a, b;
};
std::mutex g_prof_mu;
bool g_prof_on = false;
std::vector<ProfRec> g_prof_pending;
constexpr int kProfKernels = 8;
int64_t g_prof_count[kProfKernels] = {};
double g_prof_ms[kProfKernels] = {};
}  // namespace

TraceRange::TraceRange(const char *name) : pushed(quiet([&] { roctxRangePushA(name); })) {}
TraceRange::~TraceRange()
{
    if (pushed) quiet([] { roctxRangePop(); });
}

ProfScope::ProfScope(int k, hipStream_t s) : kernel(k), stream(s)
{
    std::lock_guard<std::mutex> lk(g_prof_mu);
    if (!g_prof_on) return;
    hipEvent_t e;
    if (hipEventCreate(&e) != hipSuccess) return;
    (void)hipEventRecord(e, stream);
    ev0 = e;
}

ProfScope::~ProfScope()
{
    if (!ev0) return;
    quiet([&] {
        hipEvent_t e;
        if (hipEventCreate(&e) != hipSuccess) {
            (void)hipEventDestroy((hipEvent_t)ev0);
            return;
        }
        (void)hipEventRecord(e, stream);
        std::lock_guard<std::mutex> lk(g_prof_mu);
        g_prof_pending.push_back({kernel, (hipEvent_t)ev0, e});
    });
}

// ---------------------------------------------------------------- weights

// Laplacian weights of Sec. 3.1 Eq. weightsLap.  The factorial ratio
// (n_o!)^2 / ((n_o-p)!(n_o+p)!) is accumulated as a product of p factors
// (n_o-p+i)/(n_o+i), i = 1..p.
static void laplacian_weights(int no, double h, double *w)
{
    double inv_h2 = 1.0 / (h * h);
    double s = 0.0;
    for (int q = no; q >= 1; --q) s += 1.0 / (double(q) * q);
    w[0] = -s * inv_h2;
    for (int p = 1; p <= no; ++p) {
        double ratio = 1.0;
        for (int i = 1; i <= p; ++i) ratio *= double(no - p + i) / double(no + i);
        double sign = (p & 1) ? 1.0 : -1.0;
        w[p] = 2.0 * sign * ratio / (double(p) * p) * inv_h2;
    }
    for (int p = no + 1; p <= kMaxRadius; ++p) w[p] = 0.0;
}

static bool overlaps(const void *a, size_t na, const void *b, size_t nb)
{
    if (!a || !b || na == 0 || nb == 0) return false;
    const char *pa = (const char *)a, *pb = (const char *)b;
    return pa < pb + nb && pb < pa + na;
}

static size_t block_bytes(int64_t nd, int64_t ld, int ns, int dtype)
{
    return (size_t)((int64_t)(ns - 1) * ld + nd) * elem_size(dtype);
}

static int check_block(const sparc_op *op, const void *p, int64_t ld, int ns, const char *name)
{
    if (!p) return fail(SPARC_E_ARG, std::string(name) + " is NULL");
    if (ns < 1) return fail(SPARC_E_SHAPE, "ns must be >= 1");
    if (ld < op->nd) return fail(SPARC_E_SHAPE, std::string("leading dimension of ") + name + " is below N_d");
    return SPARC_OK;
}

int append_units(const int n[3], int64_t nd, const int lo[3], const int ext[3], std::vector<int> &units,
                 std::vector<int> &pos)
{
    int cnt = 0;
    size_t loc = pos.size();
    pos.resize(loc + (size_t)ext[0] * ext[1] * ext[2]);
    for (int i = 0; i < ext[0]; ++i)
        for (int j = 0; j < ext[1]; ++j) {
            const int64_t row = (int64_t)n[2] * ((lo[1] + j) + (int64_t)n[1] * (lo[0] + i));
            const int z0 = lo[2], z1 = lo[2] + ext[2];
            for (int s = z0 / 4 * 4; s < z1; s += 4) {
                // the last unit of the grid starts 4 nodes before its end
                const int64_t first = std::max<int64_t>(0, std::min<int64_t>(row + s, nd - 4));
                int mask = 0;
                for (int z = std::max(s, z0); z < std::min(s + 4, z1); ++z, ++loc) {
                    const int b = (int)(row + z - first);
                    mask |= 1 << b;
                    pos[loc] = 4 * cnt + b;
                }
                units.push_back((int)first);
                units.push_back(mask);
                ++cnt;
            }
        }
    return cnt;
}

int launch_h_step(const sparc_op *op, int dtype, const void *yk, int64_t ldk, const void *yprev, int64_t ldp,
                  void *out, int64_t ldo, int ns, void *part, const StepCoef &c, const StepLaunch &L,
                  hipStream_t stream, const FLaunch *V)
{
    int st;
    const int nparts = op->natoms > 0 && dtype == SPARC_F32 && gather_wide(op, ns) ? 1 : kGatherSplit;
    void *tail = part;
    if (part && nparts == 1) {
        if ((st = launch_gather(op, dtype, yk, ldk, ns, part, nparts, stream))) return st;
        tail = nullptr;
    }
    if (V && V->plan >= 0)
        st = launch_fstep(op, dtype, *V, yk, ldk, yprev, ldp, out, ldo, ns, tail, c, stream);
    else
        st = launch_step_gather(op, dtype, yk, ldk, yprev, ldp, out, ldo, ns, tail, c, L, stream);
    if (st) return st;
    return launch_scatter(op, dtype, out, ldo, ns, part, nparts, c.alpha, stream);
}

}  // namespace sparc

using namespace sparc;

extern "C" {

const char *sparc_status_str(int s)
{
    switch (s) {
        case SPARC_OK: return "ok";
        case SPARC_PENDING: return "pending";
        case SPARC_E_ARG: return "invalid argument";
        case SPARC_E_SHAPE: return "inconsistent shape";
        case SPARC_E_BOUNDS: return "invalid filter bounds or degree";
        case SPARC_E_NOMEM: return "out of device memory";
        case SPARC_E_HIP: return "HIP runtime error";
        case SPARC_E_BUSY: return "reserved";
        case SPARC_E_TICKET: return "unknown ticket";
        case SPARC_E_JOB: return "job failed";
        case SPARC_E_WORKSPACE: return "workspace missing or too small";
        case SPARC_E_BREAKDOWN: return "numerical breakdown (Lanczos invariant subspace or singular M_s)";
        case SPARC_E_ALIAS: return "overlapping buffers";
    }
    return "unknown status";
}

const char *sparc_last_error(void) { return g_last_error.c_str(); }

int sparc_profile_enable(int32_t on)
{
    std::lock_guard<std::mutex> lk(g_prof_mu);
    g_prof_on = on != 0;
    return SPARC_OK;
}

int sparc_profile_reset(void)
{
    std::lock_guard<std::mutex> lk(g_prof_mu);
    for (auto &r : g_prof_pending) {
        (void)hipEventSynchronize(r.b);
        (void)hipEventDestroy(r.a);
        (void)hipEventDestroy(r.b);
    }
    g_prof_pending.clear();
    for (int k = 0; k < kProfKernels; ++k) {
        g_prof_count[k] = 0;
        g_prof_ms[k] = 0;
    }
    return SPARC_OK;
}

int sparc_profile_read(int32_t kernel, int64_t *launches, double *total_ms)
{
    if (kernel < 0 || kernel >= kProfKernels) return fail(SPARC_E_ARG, "kernel id must be 0..7");
    std::lock_guard<std::mutex> lk(g_prof_mu);
    for (auto &r : g_prof_pending) {
        if (hipEventSynchronize(r.b) != hipSuccess) return fail(SPARC_E_HIP, "event synchronisation failed");
        float ms = 0;
        (void)hipEventElapsedTime(&ms, r.a, r.b);
        g_prof_count[r.kernel] += 1;
        g_prof_ms[r.kernel] += ms;
        (void)hipEventDestroy(r.a);
        (void)hipEventDestroy(r.b);
    }
    g_prof_pending.clear();
    if (launches) *launches = g_prof_count[kernel];
    if (total_ms) *total_ms = g_prof_ms[kernel];
    return SPARC_OK;
}

int sparc_op_create(const sparc_grid *grid, const double *veff, int32_t natoms, const sparc_atom *atoms,
                    sparc_op **out)
{
    if (!grid || !veff || !out || natoms < 0 || (natoms > 0 && !atoms))
        return fail(SPARC_E_ARG, "null argument or negative atom count");
    *out = nullptr;
    for (int d = 0; d < 3; ++d)
        if (grid->n[d] < 1) return fail(SPARC_E_SHAPE, "grid extents must be >= 1");
    if (!(grid->h > 0)) return fail(SPARC_E_SHAPE, "grid spacing must be > 0");
    if (grid->radius < 1 || grid->radius > kMaxRadius) return fail(SPARC_E_SHAPE, "radius must be in 1..6");
    // one FP64 plane must stay below 2 GiB (32-bit in-plane byte offsets in the kernels)
    const int64_t plane = (int64_t)grid->n[1] * grid->n[2];
    if (plane >= (1LL << 28)) return fail(SPARC_E_SHAPE, "n[1]*n[2] must be below 2^28");
    const int64_t nd_all = (int64_t)grid->n[0] * plane;

    sparc_op *op = new (std::nothrow) sparc_op();
    if (!op) return fail(SPARC_E_NOMEM, "host allocation failed");
    auto cleanup = [&](int st) {
        sparc_op_destroy(op);
        return st;
    };
    (void)hipGetDevice(&op->device);
    for (int d = 0; d < 3; ++d) op->n[d] = grid->n[d];
    op->h = grid->h;
    op->radius = grid->radius;
    op->nd = nd_all;
    laplacian_weights(op->radius, op->h, op->w);

    const int64_t nd = op->nd;
    op->vmax = -INFINITY;
    std::vector<float> v32(nd);
    for (int64_t i = 0; i < nd; ++i) {
        op->vmax = std::max(op->vmax, veff[i]);
        v32[i] = (float)veff[i];
    }
    if (hipMalloc(&op->d_veff64, nd * sizeof(double)) != hipSuccess ||
        hipMalloc(&op->d_veff32, nd * sizeof(float)) != hipSuccess)
        return cleanup(fail(SPARC_E_NOMEM, "device allocation of V_eff failed"));
    if (hipMemcpy(op->d_veff64, veff, nd * sizeof(double), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(op->d_veff32, v32.data(), nd * sizeof(float), hipMemcpyHostToDevice) != hipSuccess)
        return cleanup(fail(SPARC_E_HIP, "copy of V_eff failed"));

    // atoms
    op->natoms = natoms;
    int64_t chi_total = 0, box_total = 0, chiu_total = 0;
    std::vector<int> units, upos;
    for (int J = 0; J < natoms; ++J) {
        const sparc_atom &A = atoms[J];
        if (A.nproj < 1 || A.nproj > kMaxProj || !A.chi || !A.gamma)
            return cleanup(fail(SPARC_E_ARG, "atom " + std::to_string(J) + ": nproj outside 1..16 or null data"));
        for (int d = 0; d < 3; ++d)
            if (A.ext[d] < 1 || A.lo[d] < 0 || A.lo[d] + A.ext[d] > grid->n[d])
                return cleanup(fail(SPARC_E_SHAPE, "atom " + std::to_string(J) + ": projector cube outside the grid"));
        AtomDev a;
        for (int d = 0; d < 3; ++d) {
            a.lo[d] = A.lo[d];
            a.ext[d] = A.ext[d];
        }
        a.nproj = A.nproj;
        a.proj0 = op->nproj_total;
        a.chi0 = chi_total;
        const int64_t nbox = (int64_t)A.ext[0] * A.ext[1] * A.ext[2];
        a.box0 = (int)box_total;
        box_total += nbox;
        // the gather's unit table and chi in its layout
        a.unit0 = (int)(units.size() / 2);
        a.nunits = append_units(op->n, op->nd, a.lo, a.ext, units, upos);
        a.chiu0 = chiu_total;
        chiu_total += (int64_t)4 * a.nunits * A.nproj;
        chi_total += nbox * A.nproj;
        op->nproj_total += A.nproj;
        op->max_nproj = std::max(op->max_nproj, A.nproj);
        op->atoms.push_back(a);
        double tr = 0, gmax = -INFINITY;
        for (int64_t i = 0; i < nbox * A.nproj; ++i) tr += A.chi[i] * A.chi[i];
        for (int p = 0; p < A.nproj; ++p) {
            op->gamma.push_back(A.gamma[p]);
            gmax = std::max(gmax, A.gamma[p]);
        }
        op->chi_trace.push_back(tr);
        op->atom_gmax.push_back(gmax);
    }
    if (box_total > 0x7fffffffLL) return cleanup(fail(SPARC_E_SHAPE, "projector cubes too large"));
    if (natoms > 0) {
        // (not zero-filled: the copies below write all of it)
        const std::unique_ptr<double[]> chi64(new (std::nothrow) double[chi_total]);
        if (!chi64) return cleanup(fail(SPARC_E_NOMEM, "host allocation of projector data failed"));
        for (int J = 0; J < natoms; ++J) {
            const sparc_atom &A = atoms[J];
            const int64_t cnt = (int64_t)A.ext[0] * A.ext[1] * A.ext[2] * A.nproj;
            std::memcpy(&chi64[op->atoms[J].chi0], A.chi, cnt * sizeof(double));
        }
        const double h3 = op->h * op->h * op->h;
        std::vector<double> hg64(op->nproj_total);
        std::vector<float> hg32(op->nproj_total);
        for (int p = 0; p < op->nproj_total; ++p) {
            hg64[p] = h3 * op->gamma[p];
            hg32[p] = (float)hg64[p];
        }
        if (hipMalloc(&op->d_atoms, natoms * sizeof(AtomDev)) != hipSuccess ||
            hipMalloc(&op->d_chi64, chi_total * sizeof(double)) != hipSuccess ||
            hipMalloc(&op->d_chi32, chi_total * sizeof(float)) != hipSuccess ||
            hipMalloc(&op->d_chiu64, chiu_total * sizeof(double)) != hipSuccess ||
            hipMalloc(&op->d_chiu32, chiu_total * sizeof(float)) != hipSuccess ||
            hipMalloc(&op->d_hg64, op->nproj_total * sizeof(double)) != hipSuccess ||
            hipMalloc(&op->d_hg32, op->nproj_total * sizeof(float)) != hipSuccess)
            return cleanup(fail(SPARC_E_NOMEM, "device allocation of projector data failed"));
        if (hipMemcpy(op->d_atoms, op->atoms.data(), natoms * sizeof(AtomDev), hipMemcpyHostToDevice) ||
            hipMemcpy(op->d_chi64, chi64.get(), chi_total * sizeof(double), hipMemcpyHostToDevice) ||
            hipMemcpy(op->d_hg64, hg64.data(), op->nproj_total * sizeof(double), hipMemcpyHostToDevice) ||
            hipMemcpy(op->d_hg32, hg32.data(), op->nproj_total * sizeof(float), hipMemcpyHostToDevice))
            return cleanup(fail(SPARC_E_HIP, "copy of projector data failed"));
        int st;
        if ((st = build_unit_chi(op, chiu_total))) return cleanup(st);
    }

    // cube-node grid offsets and the unique covered nodes with their (atom, cube index) entries
    if (natoms > 0) {
        std::vector<int> boff(box_total);
        // node << 32 | position in boff, sorted by node (positions of a node stay
        // in order): three passes of 11 bits, the nodes are below 2^31
        std::vector<uint64_t> cover(box_total), other(box_total);
        std::vector<int> atom_at(box_total);
        for (int J = 0; J < natoms; ++J) {
            const AtomDev &a = op->atoms[J];
            int loc = 0;
            for (int i = 0; i < a.ext[0]; ++i)
                for (int j = 0; j < a.ext[1]; ++j)
                    for (int k = 0; k < a.ext[2]; ++k, ++loc) {
                        const int64_t g = (int64_t)(a.lo[2] + k) + (int64_t)op->n[2] * ((a.lo[1] + j) + (int64_t)op->n[1] * (a.lo[0] + i));
                        boff[a.box0 + loc] = (int)g;
                        cover[a.box0 + loc] = (uint64_t)g << 32 | (uint64_t)(a.box0 + loc);
                        atom_at[a.box0 + loc] = J;
                    }
        }
        for (int shift = 32; shift < 64; shift += 11) {
            std::vector<size_t> start(2049, 0);
            for (uint64_t v : cover) ++start[(v >> shift & 2047) + 1];
            for (int b = 0; b < 2048; ++b) start[b + 1] += start[b];
            for (uint64_t v : cover) other[start[v >> shift & 2047]++] = v;
            cover.swap(other);
        }
        // unique nodes and their (atom, cube index) entries
        std::vector<int> pts, off;
        std::vector<std::pair<int, int>> raw;
        raw.reserve(cover.size());
        for (size_t e = 0; e < cover.size(); ++e) {
            const int g = (int)(cover[e] >> 32), at = (int)(cover[e] & 0xffffffffu), J = atom_at[at];
            if (e == 0 || g != pts.back()) {
                pts.push_back(g);
                off.push_back((int)e);
            }
            raw.push_back({J, at - op->atoms[J].box0});
        }
        off.push_back((int)cover.size());
        // scatter blocks: at most kBlock nodes touching at most kScatterSlots atoms
        std::vector<int> blk_pt{0}, blk_at{0}, blk_atoms, ent(4 * raw.size()), entu;
        const bool unit_ent = chiu_total <= 0x7fffffffLL;
        if (unit_ent) entu.resize(ent.size());
        std::vector<int> slot_of(natoms, -1);
        std::vector<int> cur;
        auto close_block = [&](int end_pt) {
            blk_pt.push_back(end_pt);
            op->nl_max_slots = std::max(op->nl_max_slots, (int)cur.size());
            for (int J : cur) {
                blk_atoms.push_back(J);
                slot_of[J] = -1;
            }
            blk_at.push_back((int)blk_atoms.size());
            cur.clear();
        };
        for (size_t pi = 0; pi < pts.size(); ++pi)
            if (off[pi + 1] - off[pi] > kScatterSlots)
                return cleanup(fail(SPARC_E_SHAPE, "more than 32 projector cubes overlap at one node"));
        for (size_t pi = 0; pi < pts.size(); ++pi) {
            int fresh = 0;
            for (int e = off[pi]; e < off[pi + 1]; ++e)
                if (slot_of[raw[e].first] < 0) ++fresh;
            const int in_block = (int)pi - blk_pt.back();
            if (in_block == kBlock || (int)cur.size() + fresh > kScatterSlots) close_block((int)pi);
            for (int e = off[pi]; e < off[pi + 1]; ++e) {
                const int J = raw[e].first;
                if (slot_of[J] < 0) {
                    slot_of[J] = (int)cur.size();
                    cur.push_back(J);
                }
                const AtomDev &a = op->atoms[J];
                const int nbox = a.ext[0] * a.ext[1] * a.ext[2];
                ent[4 * e + 0] = (int)(a.chi0 + raw[e].second);
                ent[4 * e + 1] = nbox;
                ent[4 * e + 2] = slot_of[J];
                ent[4 * e + 3] = a.nproj;
                if (unit_ent) {
                    entu[4 * e + 0] = (int)(a.chiu0 + upos[a.box0 + raw[e].second]);
                    entu[4 * e + 1] = 4 * a.nunits;
                    entu[4 * e + 2] = slot_of[J];
                    entu[4 * e + 3] = a.nproj;
                }
            }
        }
        close_block((int)pts.size());
        std::vector<int> proj(raw.size()), seg(kRedBlocks + 1);
        for (size_t e = 0; e < raw.size(); ++e) proj[e] = op->atoms[raw[e].first].proj0;
        const long long sl = red_segment(op->nd);
        for (int b = 0; b <= kRedBlocks; ++b)
            seg[b] = (int)(std::lower_bound(pts.begin(), pts.end(), b * sl,
                                            [](int x, long long y) { return (long long)x < y; }) - pts.begin());
        if (chi_total > 0x7fffffffLL) return cleanup(fail(SPARC_E_SHAPE, "projector data too large"));
        op->nl_npts = (int)pts.size();
        op->nl_nblk = (int)blk_pt.size() - 1;
        // one allocation for all of them
        std::vector<std::pair<int **, const std::vector<int> *>> at = {
            {&op->d_box_off, &boff},     {&op->d_units, &units},       {&op->d_nl_pts, &pts},
            {&op->d_nl_off, &off},       {&op->d_nl_ent, &ent},        {&op->d_nl_blk_pt, &blk_pt},
            {&op->d_nl_blk_at, &blk_at}, {&op->d_nl_blk_atoms, &blk_atoms}, {&op->d_nl_proj, &proj},
            {&op->d_nl_seg, &seg}};
        if (unit_ent) at.push_back({&op->d_nl_entu, &entu});
        size_t total = 0;
        for (auto &t : at) total += (t.second->size() + 63) / 64 * 64;
        if (hipMalloc(&op->d_tables, total * sizeof(int)) != hipSuccess)
            return cleanup(fail(SPARC_E_NOMEM, "device allocation of projector tables failed"));
        // small sets go over in one copy, large ones without a host copy of their own
        std::vector<int> all;
        const bool joint = total <= (size_t)1 << 18;
        if (joint) all.resize(total);
        size_t place = 0;
        for (auto &t : at) {
            if (joint)
                std::copy(t.second->begin(), t.second->end(), all.begin() + place);
            else if (hipMemcpy(op->d_tables + place, t.second->data(), t.second->size() * sizeof(int),
                               hipMemcpyHostToDevice) != hipSuccess)
                return cleanup(fail(SPARC_E_HIP, "copy of projector tables failed"));
            *t.first = op->d_tables + place;
            place += (t.second->size() + 63) / 64 * 64;
        }
        if (joint && hipMemcpy(op->d_tables, all.data(), total * sizeof(int), hipMemcpyHostToDevice) != hipSuccess)
            return cleanup(fail(SPARC_E_HIP, "copy of projector tables failed"));
    }
    // The copies and fills run on the null stream.  A copy from pageable memory
    // may return once the data is staged, a fill as soon as it is enqueued (the
    // API synchronisation rules of the CUDA runtime, which HIP follows), and a
    // non-blocking stream, which may use the operator next, does not wait for the
    // null stream.
    if (hipStreamSynchronize(0) != hipSuccess) return cleanup(fail(SPARC_E_HIP, "copies of the operator's data failed"));
    *out = op;
    return SPARC_OK;
}

int sparc_op_destroy(sparc_op *op)
{
    if (!op) return SPARC_OK;
    for (void *p : std::initializer_list<void *>{op->d_veff64, op->d_veff32, op->d_atoms, op->d_chi64, op->d_chi32,
                                                 op->d_hg64, op->d_hg32, op->d_tables, op->d_chiu64, op->d_chiu32,
                                                 op->d_fatoms, op->d_funits, op->d_ffun, op->d_fgamma})
        quiet([&] { (void)hipFree(p); });
    delete op;
    return SPARC_OK;
}

int64_t sparc_op_nd(const sparc_op *op) { return op ? op->nd : 0; }
int32_t sparc_op_nproj(const sparc_op *op) { return op ? op->nproj_total : 0; }

size_t sparc_workspace_bytes(const sparc_op *op, int32_t dtype, int32_t ns, int32_t which)
{
    if (!op || ns < 1 || (dtype != SPARC_F64 && dtype != SPARC_F32)) return 0;
    const size_t g = gather_bytes(op, dtype, ns);
    if (which == 0) return g;
    return g + align_up((size_t)op->nd * ns * elem_size(dtype));
}

int sparc_op_set_launch(sparc_op *op, int32_t dtype, int32_t tile_z, int32_t tile_y, int32_t chunk_x,
                        int32_t col_group, int32_t col_block)
{
    if (!op || (dtype != SPARC_F64 && dtype != SPARC_F32)) return fail(SPARC_E_ARG, "null op or bad dtype");
    if (col_block < 0 || col_block > 2) return fail(SPARC_E_ARG, "col_block must be 0, 1 or 2");
    if (tile_z <= 0 && tile_y <= 0) {
        op->tune_shape[dtype] = -1;
        op->tune_ty[dtype] = 0;
    } else {
        // patches of TY x TZ nodes offered for the dtype, and the row-pair
        // kernels' own for the grid
        int found = -1;
        for (int p = 0; p < kNumPlans; ++p)
            if (kPlanTZ[p] == tile_z && kPlanTY[p] == tile_y && vec_plan_valid(dtype, p)) found = p;
        if (found < 0 && rstep_patch(op, dtype, tile_z, tile_y)) found = kRowPair;
        if (found < 0) return fail(SPARC_E_ARG, "unsupported tile shape");
        if (col_block == 2 && (found == kRowPair || vec_max_cblk(dtype, found) < 2))
            return fail(SPARC_E_ARG, "this tile shape takes one column per workgroup");
        op->tune_shape[dtype] = found;
        op->tune_ty[dtype] = tile_y;
    }
    op->tune_chunk[dtype] = chunk_x > 0 ? chunk_x : 0;
    op->tune_group[dtype] = col_group > 0 ? col_group : 0;
    op->tune_cblk[dtype] = col_block;
    op->tune_ns[dtype] = -1;
    return SPARC_OK;
}

int sparc_step_config(const sparc_op *op, int32_t dtype, int32_t ns, int32_t *tile_z, int32_t *tile_y,
                      int32_t *chunk_x, int32_t *col_group, int32_t *col_block)
{
    if (!op || ns < 1 || (dtype != SPARC_F64 && dtype != SPARC_F32)) return fail(SPARC_E_ARG, "null op, ns < 1 or bad dtype");
    const FLaunch V = choose_vec_launch(op, dtype, ns, {});
    if (V.plan >= 0) {
        if (tile_z) *tile_z = V.plan == kRowPair ? V.tz : kPlanTZ[V.plan];
        if (tile_y) *tile_y = V.plan == kRowPair ? V.ty : kPlanTY[V.plan];
        if (chunk_x) *chunk_x = V.chunk_x;
        if (col_group) *col_group = std::min(V.cgroup, (ns + V.cblk - 1) / V.cblk);
        if (col_block) *col_block = V.cblk;
        return SPARC_OK;
    }
    StepLaunch L = choose_step_launch(op, dtype, ns);
    if (tile_z) *tile_z = kShapes[L.shape].tz;
    if (tile_y) *tile_y = kShapes[L.shape].ty();
    if (chunk_x) *chunk_x = L.chunk_x;
    if (col_group) *col_group = 1;
    if (col_block) *col_block = 1;
    return SPARC_OK;
}

int sparc_h_apply(const sparc_op *op, int32_t dtype, const void *X, int64_t ldx, void *Y, int64_t ldy, int32_t ns,
                  void *ws, size_t ws_bytes, void *stream)
{
    if (!op) return fail(SPARC_E_ARG, "op is NULL");
    if (dtype != SPARC_F64 && dtype != SPARC_F32) return fail(SPARC_E_ARG, "dtype must be SPARC_F64 or SPARC_F32");
    int st;
    if ((st = check_block(op, X, ldx, ns, "X")) || (st = check_block(op, Y, ldy, ns, "Y"))) return st;
    const size_t need = sparc_workspace_bytes(op, dtype, ns, 0);
    if (op->natoms > 0 && (!ws || ws_bytes < need)) return fail(SPARC_E_WORKSPACE, "workspace too small");
    const size_t bx = block_bytes(op->nd, ldx, ns, dtype), by = block_bytes(op->nd, ldy, ns, dtype);
    if (overlaps(X, bx, Y, by) || overlaps(X, bx, ws, need) || overlaps(Y, by, ws, need))
        return fail(SPARC_E_ALIAS, "X, Y and the workspace must not overlap");
    hipStream_t s = (hipStream_t)stream;
    StepCoef c{1.0, 0.0, 0.0, 0};
    const FLaunch V = choose_vec_launch(op, dtype, ns, {ldx, ldy});
    StepLaunch L = choose_step_launch(op, dtype, ns);
    TraceRange trace("sparc_h_apply");
    return launch_h_step(op, dtype, X, ldx, nullptr, 0, Y, ldy, ns, ws, c, L, s, &V);
}

int sparc_cheb_filter(const sparc_op *op, int32_t dtype, const void *X, int64_t ldx, void *Y, int64_t ldy,
                      int32_t ns, int32_t m, double a0, double a, double b, void *ws, size_t ws_bytes, void *stream)
{
    if (!op) return fail(SPARC_E_ARG, "op is NULL");
    if (dtype != SPARC_F64 && dtype != SPARC_F32) return fail(SPARC_E_ARG, "dtype must be SPARC_F64 or SPARC_F32");
    if (m < 1) return fail(SPARC_E_BOUNDS, "degree m must be >= 1");
    if (!(a0 < a && a < b) || !std::isfinite(a0) || !std::isfinite(b))
        return fail(SPARC_E_BOUNDS, "filter bounds must satisfy a0 < a < b");
    int st;
    if ((st = check_block(op, X, ldx, ns, "X")) || (st = check_block(op, Y, ldy, ns, "Y"))) return st;
    const size_t need = sparc_workspace_bytes(op, dtype, ns, 1);
    if (!ws || ws_bytes < need) return fail(SPARC_E_WORKSPACE, "workspace too small");
    const size_t bx = block_bytes(op->nd, ldx, ns, dtype), by = block_bytes(op->nd, ldy, ns, dtype);
    if (overlaps(X, bx, Y, by) || overlaps(X, bx, ws, need) || overlaps(Y, by, ws, need))
        return fail(SPARC_E_ALIAS, "X, Y and the workspace must not overlap");

    TraceRange trace("sparc_cheb_filter");
    hipStream_t s = (hipStream_t)stream;
    char *G = (char *)ws;
    char *W = G + gather_bytes(op, dtype, ns);
    const int64_t ldw = op->nd;

    // Y_k is written to buffer P for odd k and Q for even k, so that Y_m
    // lands in Y; Y_{k+1} overwrites Y_{k-1} in place.
    void *P = (m & 1) ? Y : (void *)W;
    void *Q = (m & 1) ? (void *)W : Y;
    const int64_t ldP = (m & 1) ? ldy : ldw;
    const int64_t ldQ = (m & 1) ? ldw : ldy;

    const double e = 0.5 * (b - a);
    const double c = 0.5 * (b + a);
    const double sigma1 = e / (a0 - c);
    const double tau = 2.0 / sigma1;
    // one kernel family for every step of the filter
    const FLaunch V = choose_vec_launch(op, dtype, ns, {ldx, ldy, ldw});
    StepLaunch L = choose_step_launch(op, dtype, ns);

    // Y_1 = (sigma_1/e)(H - cI) X
    StepCoef c1{sigma1 / e, 0.0, c, 0};
    {
        TraceRange step("filter step");
        if ((st = launch_h_step(op, dtype, X, ldx, nullptr, 0, P, ldP, ns, G, c1, L, s, &V))) return st;
    }

    double sigma = sigma1;
    for (int k = 1; k < m; ++k) {
        const double sigma_next = 1.0 / (tau - sigma);
        const void *yk = (k & 1) ? P : Q;
        const int64_t ldk = (k & 1) ? ldP : ldQ;
        const void *yprev = (k == 1) ? X : ((k & 1) ? Q : P);
        const int64_t ldp = (k == 1) ? ldx : ((k & 1) ? ldQ : ldP);
        void *out = ((k + 1) & 1) ? P : Q;
        const int64_t ldo = ((k + 1) & 1) ? ldP : ldQ;
        StepCoef ck{2.0 * sigma_next / e, sigma * sigma_next, c, 1};
        TraceRange step("filter step");
        if ((st = launch_h_step(op, dtype, yk, ldk, yprev, ldp, out, ldo, ns, G, ck, L, s, &V))) return st;
        sigma = sigma_next;
    }
    return SPARC_OK;
}

int sparc_upper_bound(const sparc_op *op, double *ub)
{
    if (!op || !ub) return fail(SPARC_E_ARG, "null argument");
    // 1D symbol of -1/2 lap_h: s(t) = -w_0 - sum_p w_p cos(p t); maximise on a
    // fine grid and add the Lipschitz bound times the grid step.
    const int N = 20000;
    double smax = -INFINITY, lip = 0;
    for (int p = 1; p <= op->radius; ++p) lip += std::fabs(op->w[p]) * p;
    for (int i = 0; i <= N; ++i) {
        const double t = M_PI * i / N;
        double s = -op->w[0];
        for (int p = 1; p <= op->radius; ++p) s -= op->w[p] * std::cos(p * t);
        smax = std::max(smax, s);
    }
    smax += lip * (M_PI / N);
    double bound = 3.0 * smax + op->vmax;
    const double h3 = op->h * op->h * op->h;
    for (int J = 0; J < op->natoms; ++J)
        if (op->atom_gmax[J] > 0) bound += h3 * op->atom_gmax[J] * op->chi_trace[J];
    *ub = bound;
    return SPARC_OK;
}

int sparc_select_bounds(const double *theta, int32_t k, int32_t nwant, double shift, double bfactor, double ubound,
                        double *a0, double *a, double *b)
{
    if (!theta || k < 1 || nwant < 1 || !a0 || !a || !b) return fail(SPARC_E_ARG, "bad arguments");
    const int iw = std::min(nwant, k) - 1;
    double A0 = theta[0], A = theta[iw] + shift, B = bfactor * theta[k - 1];
    if (ubound > 0 && ubound < B) B = ubound;
    if (!(A0 < A && A < B)) return fail(SPARC_E_BOUNDS, "Ritz values give degenerate filter bounds");
    *a0 = A0;
    *a = A;
    *b = B;
    return SPARC_OK;
}

}  // extern "C"
