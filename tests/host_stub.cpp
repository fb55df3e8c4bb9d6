// A HIP runtime, rocBLAS, rocSOLVER and roctx for the library's host code on a
// machine without a GPU: "device" memory is zeroed host memory, copies are
// memcpy, kernels and library routines do nothing.  Every call is recorded as
// one line of a log, so that tests can check what the host side asks for
// (allocations, copies, waits, launch shapes), and any call can be made to
// throw once per `stub_throw`.
#include <hip/hip_runtime.h>
#include <rocblas/rocblas.h>
#include <rocsolver/rocsolver.h>

#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <variant>

namespace {

// (made on first use: the kernels register before this unit's globals exist)
struct State {
    std::mutex mu;
    std::string log, raise;
    std::map<const void *, std::string> kernels;
};
State &st()
{
    static State *s = new State;
    return *s;
}
void (*g_d2h)(void *, const void *, size_t) = nullptr;

struct Config {
    dim3 grid, block;
    size_t lds;
    hipStream_t stream;
};
thread_local Config t_config;

// throws where stub_throw names `what`
void raise_if(const char *what)
{
    {
        std::lock_guard<std::mutex> lk(st().mu);
        if (st().raise != what) return;
    }
    const std::variant<int, double> v(1);
    (void)std::get<double>(v);
}

void note(const char *what, const char *fmt = "", ...)
{
    char text[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(text, sizeof(text), fmt, ap);
    va_end(ap);
    {
        std::lock_guard<std::mutex> lk(st().mu);
        st().log += std::string(what) + " " + text + "\n";
    }
    raise_if(what);
}

template <typename P>
P handle()
{
    return (P)std::calloc(1, 64);
}

hipError_t copy(const char *what, void *dst, const void *src, size_t n, hipMemcpyKind kind, hipStream_t s)
{
    note(what, "dst=%p src=%p bytes=%zu kind=%d stream=%p", dst, src, n, (int)kind, (void *)s);
    if (kind == hipMemcpyDeviceToHost && g_d2h)
        g_d2h(dst, src, n);
    else
        std::memcpy(dst, src, n);
    return hipSuccess;
}

hipError_t allocate(const char *what, void **p, size_t n)
{
    raise_if(what);
    *p = std::calloc(1, n ? n : 1);
    note(what, "ptr=%p bytes=%zu", *p, n);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}

}  // namespace

extern "C" {

void stub_reset()
{
    std::lock_guard<std::mutex> lk(st().mu);
    st().log.clear();
    st().raise.clear();
}
// the log, valid until the next call into the library
const char *stub_log()
{
    std::lock_guard<std::mutex> lk(st().mu);
    return st().log.c_str();
}
// every call of this name throws std::bad_variant_access from now on ("": none)
void stub_throw(const char *name)
{
    std::lock_guard<std::mutex> lk(st().mu);
    st().raise = name;
}
// device-to-host copies call f instead (null: plain copies)
void stub_d2h(void (*f)(void *, const void *, size_t)) { g_d2h = f; }

// ---------------------------------------------------------------- launches

void **__hipRegisterFatBinary(const void *) { return handle<void **>(); }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *, void *, void *, void *,
                           int *)
{
    std::lock_guard<std::mutex> lk(st().mu);
    st().kernels[f] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s)
{
    t_config = {grid, block, lds, s};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *s)
{
    *grid = t_config.grid;
    *block = t_config.block;
    *lds = t_config.lds;
    *s = t_config.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **, size_t lds, hipStream_t s)
{
    std::string name;
    {
        std::lock_guard<std::mutex> lk(st().mu);
        name = st().kernels[f];
    }
    note("hipLaunchKernel", "grid=%u,%u,%u block=%u,%u,%u lds=%zu stream=%p name=%.200s", g.x, g.y, g.z, b.x, b.y, b.z,
         lds, (void *)s, name.c_str());
    return hipSuccess;
}

// ---------------------------------------------------------------- HIP

hipError_t hipMalloc(void **p, size_t n) { return allocate("hipMalloc", p, n); }
hipError_t hipMallocAsync(void **p, size_t n, hipStream_t) { return allocate("hipMallocAsync", p, n); }
hipError_t hipFree(void *p)
{
    if (p) note("hipFree", "ptr=%p", p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipFreeAsync(void *p, hipStream_t s)
{
    note("hipFreeAsync", "ptr=%p stream=%p", p, (void *)s);
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind k) { return copy("hipMemcpy", d, s, n, k, nullptr); }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t st)
{
    return copy("hipMemcpyAsync", d, s, n, k, st);
}
hipError_t hipMemset(void *d, int v, size_t n)
{
    note("hipMemset", "dst=%p bytes=%zu", d, n);
    std::memset(d, v, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t)
{
    note("hipMemsetAsync", "dst=%p bytes=%zu", d, n);
    std::memset(d, v, n);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s)
{
    note("hipStreamSynchronize", "stream=%p", (void *)s);
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned)
{
    raise_if("hipStreamCreateWithFlags");
    *s = handle<hipStream_t>();
    note("hipStreamCreateWithFlags", "stream=%p", (void *)*s);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s)
{
    note("hipStreamDestroy", "stream=%p", (void *)s);
    std::free(s);
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g)
{
    *g = handle<hipGraph_t>();
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t)
{
    *e = handle<hipGraphExec_t>();
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t g)
{
    std::free(g);
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t e)
{
    std::free(e);
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e)
{
    *e = handle<hipEvent_t>();
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e)
{
    std::free(e);
    return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t)
{
    note("hipEventQuery");
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t)
{
    note("hipEventRecord");
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t)
{
    *ms = 1.0f;
    return hipSuccess;
}
hipError_t hipGetDevice(int *d)
{
    *d = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int)
{
    note("hipSetDevice");
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int)
{
    *v = 256;
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t)
{
    *n = 2;
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *)
{
    static char scratch[16 << 20];
    *p = scratch;
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "hip error"; }

// ---------------------------------------------------------------- libraries

int roctxRangePushA(const char *)
{
    note("roctxRangePushA");
    return 0;
}
int roctxRangePop()
{
    note("roctxRangePop");
    return 0;
}
rocblas_status rocblas_create_handle(rocblas_handle *h)
{
    *h = handle<rocblas_handle>();
    note("rocblas_create_handle");
    return rocblas_status_success;
}
rocblas_status rocblas_destroy_handle(rocblas_handle h)
{
    note("rocblas_destroy_handle");
    std::free(h);
    return rocblas_status_success;
}
rocblas_status rocblas_set_stream(rocblas_handle, hipStream_t)
{
    note("rocblas_set_stream");
    return rocblas_status_success;
}
rocblas_status rocblas_set_atomics_mode(rocblas_handle, rocblas_atomics_mode) { return rocblas_status_success; }
const char *rocblas_status_to_string(rocblas_status) { return "rocblas status"; }
rocblas_status rocblas_dtrsm(rocblas_handle, rocblas_side, rocblas_fill, rocblas_operation, rocblas_diagonal,
                             rocblas_int, rocblas_int, const double *, const double *, rocblas_int, double *, rocblas_int)
{
    note("rocblas_dtrsm");
    return rocblas_status_success;
}
rocblas_status rocblas_dgemm(rocblas_handle, rocblas_operation, rocblas_operation, rocblas_int, rocblas_int, rocblas_int,
                             const double *, const double *, rocblas_int, const double *, rocblas_int, const double *,
                             double *, rocblas_int)
{
    note("rocblas_dgemm");
    return rocblas_status_success;
}
rocblas_status rocblas_sgemm(rocblas_handle, rocblas_operation, rocblas_operation, rocblas_int, rocblas_int, rocblas_int,
                             const float *, const float *, rocblas_int, const float *, rocblas_int, const float *,
                             float *, rocblas_int)
{
    note("rocblas_sgemm");
    return rocblas_status_success;
}
rocblas_status rocsolver_dpotrf(rocblas_handle, const rocblas_fill, const rocblas_int, double *, const rocblas_int,
                                rocblas_int *)
{
    note("rocsolver_dpotrf");
    return rocblas_status_success;
}
rocblas_status rocsolver_dsyevd(rocblas_handle, const rocblas_evect, const rocblas_fill, const rocblas_int, double *,
                                const rocblas_int, double *, double *, rocblas_int *)
{
    note("rocsolver_dsyevd");
    return rocblas_status_success;
}

}  // extern "C"
