// kernels_small.hip -- the whole of Algorithm 1 for a small system in one
// workgroup (gfx950).
//
// p lives in LDS (every row may read any entry); thread t of NT owns rows
// t, t + NT, ... and keeps their x, r, q and p in registers.  The launch reads x0
// from the caller's x, writes the solution there, recomputes the true
// residual b - A x at the end and leaves every result in the device state,
// so a solve is one launch and one read-back of that state.
#include <hip/hip_runtime.h>
#include <math.h>

#include "cgmi_internal.h"

namespace cgmi {

namespace {

constexpr int kWave = kWaveSize;
constexpr int kSmallRows = 4096;   // rows of a workgroup at most

// One DPP move of a double (both 32-bit halves with the same lane pattern).
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ double readlane_f64(double v, int lane) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// Sum over the wave, the same value in every lane, without LDS: a butterfly
// inside each row of 16 lanes (swap neighbours, swap pairs, mirror the half
// rows, mirror the row) leaves every lane with its row's sum; the four row
// sums are then read as scalars and added in a fixed order.
__device__ __forceinline__ double row_allsum_dpp(double v) {
    v += dpp_f64<0xB1>(v);   // quad_perm [1,0,3,2]
    v += dpp_f64<0x4E>(v);   // quad_perm [2,3,0,1]
    v += dpp_f64<0x141>(v);  // row_half_mirror
    v += dpp_f64<0x140>(v);  // row_mirror
    return v;
}
__device__ __forceinline__ double wave_allsum_dpp(double v) {
    v = row_allsum_dpp(v);
    return (readlane_f64(v, 0) + readlane_f64(v, 16)) + (readlane_f64(v, 32) + readlane_f64(v, 48));
}

// Every thread gets the workgroup sum after ONE barrier: each wave posts its
// sum, then every lane reads one of the kSmallWaves posts and the rows of 16
// lanes sum them by DPP moves, all in the same order (so all threads hold
// bitwise the same value and branch alike).  Consecutive calls alternate
// between the two halves of red: a wave can only overwrite a half after the
// next call's barrier, which every thread reaches after it has read that half.
template <int NT>
__device__ __forceinline__ double small_allsum(double v, double (*red)[NT / kWave], int &half) {
    constexpr int waves = NT / kWave;
    static_assert(waves <= 16, "one post per lane of a row");
    v = wave_allsum_dpp(v);
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    if (lane == 0) red[half][w] = v;
    __syncthreads();
    const double s = row_allsum_dpp((lane & 15) < waves ? red[half][lane & 15] : 0.0);
    half ^= 1;
    return s;
}

// Row storage of a thread's RPT rows.  W > 0: rows of at most W entries held
// in registers for the whole solve (byte offsets of the columns in LDS, below
// 2^16 here, packed two to a register); slots past a row's length hold column = the row itself
// and value 0, which leaves the row's sum unchanged, so the entries are
// summed in CSR order as the CSR variant does.  W == 0: the row bounds in
// registers, columns and values read from memory at every product.
template <int NT, int RPT, int W>
struct SmallRows {
    static_assert(kSmallRows * sizeof(double) <= 65536, "packed 16-bit offsets");
    static constexpr int WP = (W + 1) / 2;
    uint32_t colp[RPT][WP];
    double a[RPT][W];
    __device__ void load(int32_t n, const int32_t *rp, const int32_t *ci, const double *val) {
        const int t = threadIdx.x;
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            const int i = t + j * NT;
            const int32_t beg = i < n ? rp[i] : 0;
            const int32_t len = i < n ? rp[i + 1] - beg : 0;
            const uint32_t self = i < n ? (uint32_t)i : 0u;
#pragma unroll
            for (int e = 0; e < WP; ++e) colp[j][e] = 0;
#pragma unroll
            for (int e = 0; e < W; ++e) {
                const uint32_t c = e < len ? (uint32_t)ci[beg + e] : self;
                colp[j][e / 2] |= (c * 8u) << (16 * (e & 1));
                a[j][e] = e < len ? val[beg + e] : 0.0;
            }
        }
    }
    template <class Get>
    __device__ __forceinline__ double dot(int j, Get get) const {
        double s = 0.0;
#pragma unroll
        for (int e = 0; e < W; ++e)
            s = fma(a[j][e], get(e & 1 ? colp[j][e / 2] >> 16 : colp[j][e / 2] & 0xFFFFu), s);
        return s;
    }
};

template <int NT, int RPT>
struct SmallRows<NT, RPT, 0> {
    int32_t r0[RPT], r1[RPT];
    const int32_t *ci;
    const double *val;
    __device__ void load(int32_t n, const int32_t *rp, const int32_t *ci_, const double *val_) {
        ci = ci_;
        val = val_;
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            const int i = threadIdx.x + j * NT;
            r0[j] = i < n ? rp[i] : 0;
            r1[j] = i < n ? rp[i + 1] : 0;
        }
    }
    template <class Get>
    __device__ __forceinline__ double dot(int j, Get get) const {
        double s = 0.0;
        for (int k = r0[j]; k < r1[j]; ++k) s = fma(val[k], get((uint32_t)ci[k] * 8u), s);
        return s;
    }
};

template <int NT, int RPT, int W>
__global__ __launch_bounds__(NT) void k_cg_small(int32_t n, const int32_t *__restrict__ rp,
                                                            const int32_t *__restrict__ ci,
                                                            const double *__restrict__ val,
                                                            const double *__restrict__ b,
                                                            double *__restrict__ x, double tol,
                                                            int32_t maxit, DevState *__restrict__ st) {
    extern __shared__ double s_p[];
    __shared__ double red[2][NT / kWave];
    int half = 0;
    const int t = threadIdx.x;
    SmallRows<NT, RPT, W> A;
    A.load(n, rp, ci, val);
    double xr[RPT], rr[RPT], qq[RPT], pr[RPT];
    double acc_r = 0.0, acc_b = 0.0;
    // r = b - A x0, p = r, rho = r^T r, bb = b^T b
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        const int i = t + j * NT;
        xr[j] = rr[j] = 0.0;
        if (i < n) {
            const double s = A.dot(j, [&](uint32_t c) { return *reinterpret_cast<const double *>(reinterpret_cast<const char *>(x) + c); });
            const double bi = b[i];
            xr[j] = x[i];
            rr[j] = bi - s;
            acc_r = fma(rr[j], rr[j], acc_r);
            acc_b = fma(bi, bi, acc_b);
        }
        s_p[i] = pr[j] = rr[j];
    }
    double rho = small_allsum<NT>(acc_r, red, half);
    const double bb = small_allsum<NT>(acc_b, red, half);
    if (bb == 0.0) {
        // b = 0: the solution is x = 0
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            const int i = t + j * NT;
            if (i < n) x[i] = 0.0;
        }
        if (t == 0) {
            st->iter = 0;
            st->done = kDoneConverged;
            st->rho[0] = st->rr = st->bb = st->rr_true = 0.0;
        }
        return;
    }
    const double bnorm = sqrt(bb);
    // far above the limit (by more than all rounding here) the test needs no
    // square root, which every wave would wait for
    const double far = tol * bnorm * (tol * bnorm) * (1.0 + 1e-12) + 1e-300;
    auto stopped = [&](double rr) { return !(rr > far) && (sqrt(rr) < tol * bnorm || rr == 0.0); };
    int status = kDoneMaxit;
    int k = 0;
    for (k = 0; k < maxit; ++k) {
        if (stopped(rho)) {
            status = kDoneConverged;
            break;
        }
        // (rows past the end hold zeros in every vector and take part, so that
        // no branch parts the loads of one row from the next one's)
        double acc = 0.0;
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            qq[j] = A.dot(j, [&](uint32_t c) { return *reinterpret_cast<const double *>(reinterpret_cast<const char *>(s_p) + c); });
            acc = fma(pr[j], qq[j], acc);
        }
        const double pq = small_allsum<NT>(acc, red, half);
        if (!(pq > 0.0) || !isfinite(pq)) {
            status = kDoneBreakdown;
            break;
        }
        const double alpha = rho / pq;
        acc = 0.0;
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            xr[j] = fma(alpha, pr[j], xr[j]);
            rr[j] = fma(-alpha, qq[j], rr[j]);
            acc = fma(rr[j], rr[j], acc);
        }
        const double rho_new = small_allsum<NT>(acc, red, half);
        const double beta = rho_new / rho;
        rho = rho_new;
#pragma unroll
        for (int j = 0; j < RPT; ++j) s_p[t + j * NT] = pr[j] = fma(beta, pr[j], rr[j]);
        __syncthreads();
    }
    if (status == kDoneMaxit && stopped(rho)) status = kDoneConverged;
    // the solution to the caller, and into LDS for the true residual b - A x
    // (every read of p has passed a barrier: the loop top follows one, a
    // breakdown follows the p^T q sum)
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        const int i = t + j * NT;
        if (i < n) {
            x[i] = xr[j];
            s_p[i] = xr[j];
        }
    }
    __syncthreads();
    double acc_t = 0.0;
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        const int i = t + j * NT;
        if (i < n) {
            // rows read once more from memory, so the registers holding them
            // are free after the loop; the same CSR order
            double s = 0.0;
            for (int kk = rp[i]; kk < rp[i + 1]; ++kk) s = fma(val[kk], s_p[ci[kk]], s);
            const double rv = b[i] - s;
            acc_t = fma(rv, rv, acc_t);
        }
    }
    const double rr_true = small_allsum<NT>(acc_t, red, half);
    if (t == 0) {
        st->iter = k;
        st->done = status;
        st->rho[0] = rho;
        st->rr = rho;
        st->bb = bb;
        st->rr_true = rr_true;
    }
}

}  // namespace

int small_path_max_rows() {
    static int cached = -1;
    if (cached < 0) {
        int dev = 0;
        hipDeviceProp_t prop;
        size_t lds = 64 * 1024;
        if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess)
            lds = prop.sharedMemPerBlock;
        const int by_lds = (int)((lds > 1024 ? lds - 1024 : 0) / sizeof(double));
        cached = by_lds < kSmallRows ? by_lds : kSmallRows;
    }
    return cached;
}

hipError_t launch_cg_small(int32_t n, const int32_t *rp, const int32_t *ci, const double *val,
                           const double *b, double *x, double tol, int32_t maxit, DevState *st,
                           int32_t max_row_len, hipStream_t s) {
    if (n <= 0 || n > small_path_max_rows() || max_row_len < 0) return hipErrorInvalidValue;
    const int L = max_row_len;
#define CGMI_SMALL(NT, R, W)                                                                                        \
    if (n <= NT * R && (W == 0 || L <= W)) {                                                                        \
        hipLaunchKernelGGL((k_cg_small<NT, R, W>), dim3(1), dim3(NT), sizeof(double) * NT * R, s, n, rp, ci, val, b, \
                           x, tol, maxit, st);                                                                      \
        return hipGetLastError();                                                                                   \
    }
    // register-resident rows where R x W entries fit beside the vectors: 512
    // threads of twice the registers, with fewer waves at the three barriers of
    // an iteration, instead of 1024 (us per iteration: 20^2 0.9 against 1.5,
    // 45^2 1.3 against 1.6, 64^2 1.6 against 1.8, and 15^3, whose rows do not
    // fit the registers of 1024 threads, 1.8 against 7.6)
    CGMI_SMALL(512, 1, 8)
    CGMI_SMALL(512, 1, 20)
    CGMI_SMALL(512, 2, 8)
    CGMI_SMALL(512, 2, 20)
    CGMI_SMALL(512, 4, 8)
    CGMI_SMALL(512, 4, 12)
    CGMI_SMALL(512, 8, 5)
    CGMI_SMALL(512, 8, 7)
    // rows read from memory: more waves have more reads in flight (4000 random
    // rows of 13 entries: 49 against 57 with 512)
    CGMI_SMALL(1024, 1, 0)
    CGMI_SMALL(1024, 2, 0)
    CGMI_SMALL(1024, 4, 0)
#undef CGMI_SMALL
    return hipErrorInvalidValue;
}

}  // namespace cgmi
