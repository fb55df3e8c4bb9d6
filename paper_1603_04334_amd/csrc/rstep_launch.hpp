// Launch code of the row-pair step kernels, instantiated per storage type,
// LDS row pitch and row kind in rstep_*.hip (separate translation units, so
// the kernel variants compile in parallel).
#pragma once

#include "nonlocal_kernel.hpp"
#include "rstep_kernel.hpp"

namespace sparc {

constexpr int kRThreads = 512;  // two waves per SIMD: up to 256 registers for two queues

// the first a.nblocks workgroups run the step, the others blockDim/256 gather
// items each (see fstep_kernel)
template <typename T, int PITCH, int NH, bool PREV, bool STREAM, int RAG>
__global__ void __launch_bounds__(kRThreads)
    rstep_kernel(const RStepArgs<T> a, const GatherArgs<T, T> g, int natoms, int ncb, int nitems)
{
    extern __shared__ __align__(16) char rstep_lds[];
    if ((int)blockIdx.x >= a.nblocks) {
        typedef T Tile[4][16][16];
        Tile *tile = (Tile *)rstep_lds;
        const int G = blockDim.x / 256, sub = threadIdx.x >> 8;
        const int item = ((int)blockIdx.x - a.nblocks) * G + sub;
        if (sub < G && item < nitems)
            gather_item<T, T>(g, item % natoms, (item / natoms) % ncb, item / (natoms * ncb), tile[sub],
                              threadIdx.x & 255);
        else
            __syncthreads();
        return;
    }
    RStep<T, PITCH, NH, PREV, STREAM, RAG> k(a);
    k.run(blockIdx.x, (T *)rstep_lds);
}

template <typename T, int PITCH, int RAG>
int rstep_dispatch(const RStepArgs<T> &a, const GatherArgs<T, T> &g, int natoms, int ncb, int nitems, int ngb,
                   int nthreads, int nh, bool prev, bool strm, hipStream_t s)
{
    const dim3 grid(a.nblocks + ngb), b(nthreads);
    const size_t lds = std::max<size_t>(2 * (size_t)(a.ty + 2 * kMaxRadius) * PITCH * sizeof(T),
                                        ngb > 0 ? (size_t)(nthreads / 256) * 1024 * sizeof(T) : 0);
#define SPARC_RS(H, P, S) \
    hipLaunchKernelGGL((rstep_kernel<T, PITCH, H, P, S, RAG>), grid, b, lds, s, a, g, natoms, ncb, nitems)
#define SPARC_RS_H(P, S)         \
    do {                         \
        if (nh == 1)             \
            SPARC_RS(1, P, S);   \
        else                     \
            SPARC_RS(2, P, S);   \
    } while (0)
    if (prev && strm)
        SPARC_RS_H(true, true);
    else if (prev)
        SPARC_RS_H(true, false);
    else if (strm)
        SPARC_RS_H(false, true);
    else
        SPARC_RS_H(false, false);
#undef SPARC_RS_H
#undef SPARC_RS
    SPARC_HIP(hipGetLastError());
    return SPARC_OK;
}

#define SPARC_RSTEP_DECL(name, T)                                                                              \
    int name(const RStepArgs<T> &, const GatherArgs<T, T> &, int, int, int, int, int, int, bool, bool, hipStream_t)
SPARC_RSTEP_DECL(rstep_f32_p112, float);
SPARC_RSTEP_DECL(rstep_f32_p112_r1, float);
SPARC_RSTEP_DECL(rstep_f32_p112_r2, float);
SPARC_RSTEP_DECL(rstep_f32_p112_r3, float);
SPARC_RSTEP_DECL(rstep_f32_p176, float);
SPARC_RSTEP_DECL(rstep_f32_p176_r1, float);
SPARC_RSTEP_DECL(rstep_f32_p176_r2, float);
SPARC_RSTEP_DECL(rstep_f32_p176_r3, float);
SPARC_RSTEP_DECL(rstep_f64_p44, double);
SPARC_RSTEP_DECL(rstep_f64_p44_r1, double);
SPARC_RSTEP_DECL(rstep_f64_p108, double);
SPARC_RSTEP_DECL(rstep_f64_p108_r1, double);

}  // namespace sparc
