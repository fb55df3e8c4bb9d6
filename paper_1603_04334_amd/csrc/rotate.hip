// Subspace rotation out = Y Q of blocks of 17 to 192 (FP64) or 224 (FP32)
// columns on the matrix cores (Sec. 3.4, Eq. OrbitalTransformation).
//
// Design.  Q (half of its columns from 129 on) stays in LDS for the whole
// launch, one workgroup of eight waves per CU, up to 64 columns three of four
// waves.  A wave takes 32 (FP64) or 64 (FP32) points and all columns of the
// panel: it streams Y once, column by column, 16 bytes per lane straight into
// the matrix instructions' operand (four loads in flight), and writes every
// output line once.  The output column is the row of the matrix product, so
// that a lane holds neighbouring points of it and stores 16 bytes.  The sum
// over the columns of Y runs in column order.
//
// What bounds it: the reads and writes of the block up to about 64 columns, from
// there the loads a wave has in flight beside its sums, then the matrix cores.
// 96^3 points, against the scalar kernel (up to 32 FP64, 64 FP32 columns) or a
// rocBLAS GEMM with a padded copy of Q: FP64 x 32 105 -> 72 us, x 64 284 -> 194,
// x 128 0.530 -> 0.509 ms, x 192 1.33 -> 1.06 ms; FP32 x 65 294 -> 105 us,
// x 128 0.297 -> 0.287 ms, x 224 0.970 -> 0.804 ms.  Wider blocks stay with the
// GEMM: FP32 x 256 0.97 ms here 1.04; FP64 x 208 does not fit in LDS.
#include <algorithm>

#include "nonlocal_kernel.hpp"

namespace sparc {
namespace {

constexpr int kRotAhead = 4;  // loads of Y in flight

constexpr int rot_waves(int ncb) { return ncb <= 4 ? 4 : 8; }  // waves per workgroup

template <typename T, int NCB, int P>
struct RotPanel {
    static constexpr int K = 16 * NCB * P;  // columns of Y at most
    // row stride of Q's columns in LDS: 2 (FP64) or 4 (FP32) times an odd number
    // of values puts the 16 columns x 4 rows of an operand in distinct banks
    static constexpr int S = sizeof(T) == 8 ? K + 2 : K + 4 * (K / 4 % 2 == 0);
};

template <typename T, int NCB, int P>
__global__ void __launch_bounds__(64 * rot_waves(NCB), NCB <= 4 ? 3 : 2)
    rotate_mfma_kernel(const T *__restrict__ Y, long long ldy, const double *__restrict__ Q, T *__restrict__ out,
                       long long ldo, long long nd, int ns, bool lines)
{
    constexpr int S = RotPanel<T, NCB, P>::S, W = rot_waves(NCB);
    constexpr int VP = 16 / sizeof(T);  // points per lane
    typedef T V __attribute__((ext_vector_type(VP)));
    typedef T VU __attribute__((ext_vector_type(VP), aligned(sizeof(T))));
    __shared__ T q[16 * NCB * S];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, li = lane & 15, lk = lane >> 4;
    const int c0 = blockIdx.y * 16 * NCB, k4 = (ns + 3) / 4 * 4;
    for (int c = wave; c < 16 * NCB; c += W)
        for (int k = lane; k < k4; k += 64)
            q[c * S + k] = c0 + c < ns && k < ns ? (T)Q[(long long)(c0 + c) * ns + k] : T(0);
    __syncthreads();
    const long long nblk = (nd + 16 * VP - 1) / (16 * VP);
    for (long long blk = (long long)blockIdx.x * W + wave; blk < nblk; blk += (long long)gridDim.x * W) {
        // the last block's lanes past the end repeat the block's last points
        const long long x = min(blk * 16 * VP + li * VP, nd - VP);
        const T *y0 = Y + x;
        auto load = [&](int k) -> V { return *(const VU *)(y0 + min(k, ns - 1) * ldy); };
        T acc[NCB][VP][4] = {};
        V buf[kRotAhead];
#pragma unroll
        for (int d = 0; d < kRotAhead; ++d)
            buf[d] = load(4 * d + lk);
        for (int k0 = 0; k0 < k4; k0 += 4 * kRotAhead) {
#pragma unroll
            for (int d = 0; d < kRotAhead; ++d) {
                const int k = k0 + 4 * d;
                if (k >= k4) break;
                const V y = k + lk < ns ? buf[d] : V(0);
                buf[d] = load(k + 4 * kRotAhead + lk);
                T a[NCB];
#pragma unroll
                for (int c = 0; c < NCB; ++c) a[c] = q[(16 * c + li) * S + k + lk];
#pragma unroll
                for (int c = 0; c < NCB; ++c)
#pragma unroll
                    for (int b = 0; b < VP; ++b) mfma_16x16x4(a[c], (T)y[b], acc[c][b]);
            }
        }
#pragma unroll
        for (int c = 0; c < NCB; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int col = c0 + 16 * c + acc_row<T>(lane, r);
                if (col >= ns) continue;
                VU v;
#pragma unroll
                for (int b = 0; b < VP; ++b) v[b] = acc[c][b][r];
                VU *p = (VU *)(out + col * ldo + x);
                if (lines)
                    __builtin_nontemporal_store(v, p);
                else
                    *p = v;
            }
    }
}

template <typename T, int NCB, int P>
void launch_t(const T *Y, long long ldy, const double *Q, T *out, long long ldo, long long nd, int ns, hipStream_t s)
{
    // as many workgroups as are resident, evened out over their rounds
    constexpr int W = rot_waves(NCB), per_cu = NCB <= 4 ? 3 : 1;
    constexpr int pts = 16 * (16 / sizeof(T));
    const long long nblk = (nd + pts - 1) / pts, slots = 256 * per_cu / P * W;
    const long long rounds = (nblk + slots - 1) / slots;
    const unsigned gx = (unsigned)((nblk + W * rounds - 1) / (W * rounds));
    // columns that start on a 128-byte line are written past the caches in whole
    // lines (96^3 x 33 FP64 102 -> 77 us); others leave it to the cache to join
    // the halves (95^3 x 128: 0.575 ms, past the caches 0.676)
    const bool lines = ((size_t)out | (size_t)ldo * sizeof(T)) % 128 == 0;
    hipLaunchKernelGGL((rotate_mfma_kernel<T, NCB, P>), dim3(gx, P), dim3(64 * W), 0, s, Y, ldy, Q, out, ldo, nd, ns,
                       lines);
}

template <typename T>
bool launch_any(const T *Y, long long ldy, const double *Q, T *out, long long ldo, long long nd, int ns, hipStream_t s)
{
    if (nd < (long long)(16 / sizeof(T))) return false;  // a lane's points
    const int nb = (ns + 15) / 16;
    switch (nb) {
        case 2: launch_t<T, 2, 1>(Y, ldy, Q, out, ldo, nd, ns, s); return true;
        case 3: launch_t<T, 3, 1>(Y, ldy, Q, out, ldo, nd, ns, s); return true;
        case 4: launch_t<T, 4, 1>(Y, ldy, Q, out, ldo, nd, ns, s); return true;
        case 5: launch_t<T, 5, 1>(Y, ldy, Q, out, ldo, nd, ns, s); return true;
        case 6: launch_t<T, 6, 1>(Y, ldy, Q, out, ldo, nd, ns, s); return true;
        case 7: launch_t<T, 7, 1>(Y, ldy, Q, out, ldo, nd, ns, s); return true;
        case 8: launch_t<T, 8, 1>(Y, ldy, Q, out, ldo, nd, ns, s); return true;
        case 9:
        case 10: launch_t<T, 5, 2>(Y, ldy, Q, out, ldo, nd, ns, s); return true;
        case 11:
        case 12: launch_t<T, 6, 2>(Y, ldy, Q, out, ldo, nd, ns, s); return true;
        default: break;
    }
    if constexpr (sizeof(T) == 4) {
        switch (nb) {
            case 13:
            case 14: launch_t<T, 7, 2>(Y, ldy, Q, out, ldo, nd, ns, s); return true;
            default: break;
        }
    }
    return false;
}

}  // namespace

bool launch_rotate_mfma(int dtype, const void *Y, int64_t ldy, const double *Q, void *out, int64_t ldo, int64_t nd,
                        int ns, hipStream_t s)
{
    if (dtype == SPARC_F64) return launch_any((const double *)Y, ldy, Q, (double *)out, ldo, nd, ns, s);
    return launch_any((const float *)Y, ldy, Q, (float *)out, ldo, nd, ns, s);
}

}  // namespace sparc
