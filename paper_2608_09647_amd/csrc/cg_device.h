// Device helpers shared by the SpMV and vector kernels: workgroup sums, the
// in-order sums of a producer kernel's partials, the stop test, and an SpMV
// row's epilogue.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>

#include "cgmi_internal.h"

namespace cgmi {
namespace {

constexpr int kWave = kWaveSize;
constexpr int kWavesPerBlock = kBlock / kWave;

enum { kFlagCheckDone = 1, kFlagFirstIter = 2 };

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_down(v, o, kWave);
    return v;
}

// Sum over the workgroup; the result is valid in thread 0.  sh: NT/64 doubles.
template <int NT>
__device__ __forceinline__ double block_sum(double v, double *sh) {
    v = wave_sum(v);
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    if (lane == 0) sh[w] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0) {
        s = sh[0];
#pragma unroll
        for (int i = 1; i < NT / kWave; ++i) s += sh[i];
    }
    __syncthreads();
    return s;
}

// Every thread of the workgroup gets the sum.
template <int NT>
__device__ __forceinline__ double block_allsum(double v, double *sh, double *bc) {
    double s = block_sum<NT>(v, sh);
    if (threadIdx.x == 0) *bc = s;
    __syncthreads();
    s = *bc;
    __syncthreads();
    return s;
}

// This thread's share of a producer kernel's partials: entries t, t + kBlock,
// t + 2 kBlock, ... added in that order.  The loads of eight entries are
// issued together, so the sum costs one memory round trip per 8 kBlock
// partials instead of one per entry.
__device__ __forceinline__ double thread_partials(const Partials &P) {
    double v = 0.0;
    for (int base = threadIdx.x; base < P.count; base += 8 * kBlock) {
        double t[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = base + u * kBlock;
            t[u] = i < P.count ? P.v[i] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (base + u * kBlock < P.count) v += t[u];
    }
    return v;
}

// Sum of a producer kernel's partials in a fixed order (same in every workgroup).
__device__ __forceinline__ double reduce_partials(const Partials &P, double *sh, double *bc) {
    return block_allsum<kBlock>(thread_partials(P), sh, bc);
}

// Two such sums with one set of workgroup barriers, each in the order of
// reduce_partials; the loads of both arrays are issued together.
// sh: 2 kBlock/64 doubles; bc: 2 doubles.
__device__ __forceinline__ void reduce_partials2(const Partials &P0, const Partials &P1, double *sh,
                                                 double *bc, double &s0, double &s1) {
    constexpr int NW = kBlock / kWave;
    double a0 = 0.0, a1 = 0.0;
    const int cmax = max(P0.count, P1.count);
    for (int base = threadIdx.x; base < cmax; base += 8 * kBlock) {
        double t0[8], t1[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = base + u * kBlock;
            t0[u] = i < P0.count ? P0.v[i] : 0.0;
            t1[u] = i < P1.count ? P1.v[i] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = base + u * kBlock;
            if (i < P0.count) a0 += t0[u];
            if (i < P1.count) a1 += t1[u];
        }
    }
    const double v0 = wave_sum(a0);
    const double v1 = wave_sum(a1);
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    if (lane == 0) {
        sh[w] = v0;
        sh[NW + w] = v1;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double a = sh[0], b = sh[NW];
#pragma unroll
        for (int i = 1; i < NW; ++i) {
            a += sh[i];
            b += sh[NW + i];
        }
        bc[0] = a;
        bc[1] = b;
    }
    __syncthreads();
    s0 = bc[0];
    s1 = bc[1];
    __syncthreads();
}

__device__ __forceinline__ bool stop_test(double rho, double bb, double tol) {
    return sqrt(rho) < tol * sqrt(bb) || rho == 0.0;
}

__device__ __forceinline__ bool is_block0_thread0() { return blockIdx.x == 0 && threadIdx.x == 0; }

// T: float64, or float32 for the inner solve of mixed precision.
template <class T>
struct SpmvArgs {
    const T *__restrict__ p;      // gathered vector (full length)
    T *__restrict__ q;            // output rows (local)
    const T *__restrict__ p_own;  // p at the block's own rows (dot)
    const T *__restrict__ b;      // residual mode: right-hand side (local)
    T *__restrict__ p_dst;        // residual mode: copy of r (local)
};

template <class T> __device__ __forceinline__ const T *csr_vals(const CsrDev &A);
template <> __device__ __forceinline__ const double *csr_vals<double>(const CsrDev &A) { return A.val; }
template <> __device__ __forceinline__ const float *csr_vals<float>(const CsrDev &A) { return A.val32; }
template <class T> __device__ __forceinline__ const T *sell_vals(const CsrDev &A);
template <> __device__ __forceinline__ const double *sell_vals<double>(const CsrDev &A) { return A.sell_val; }
template <> __device__ __forceinline__ const float *sell_vals<float>(const CsrDev &A) { return A.sell_val32; }

// Dot contributions and residual norms are always accumulated in float64.
template <int MODE, class T>
__device__ __forceinline__ void emit_row(const SpmvArgs<T> &a, int row, T s, double &acc0,
                                         double &acc1) {
    if (MODE == kSpmvResidual) {
        const T bv = a.b[row];
        const T rv = bv - s;
        a.q[row] = rv;
        a.p_dst[row] = rv;
        acc0 = fma((double)rv, (double)rv, acc0);
        acc1 = fma((double)bv, (double)bv, acc1);
    } else if (MODE == kSpmvAccum) {
        a.q[row] = a.q[row] + s;
    } else {
        a.q[row] = s;
        if (MODE == kSpmvDot) acc0 = fma((double)a.p_own[row], (double)s, acc0);
    }
}

// s + c x with the product rounded first.
__device__ __forceinline__ double add_rounded(double s, double c, double x) {
#pragma clang fp contract(off)
    return s + c * x;
}

}  // namespace
}  // namespace cgmi
