// kernels_staged.hip -- SpMV on staged column segments, for rows whose
// columns scatter over the whole vector (gfx950).
//
// A gather of a scattered column costs an L2 request of its own however few
// bytes it needs: about 157 G gathers/s on the whole GPU at best.  Here no
// gather leaves the compute unit.  A workgroup of 16 waves owns a block of
// consecutive rows and a group of the vector's segments; it keeps the rows'
// sums (float64) in LDS, stages one segment after the other there with
// full-width loads (two buffers, the next segment on its way in registers
// while the current one is used) and multiplies the block's entries of that
// segment.  With G groups every segment is staged by 1/G of the workgroups,
// and a second kernel adds the G sums of each row and ends the mode (the dot
// product, the residual, the stop test of iteration 0).  G is as large as
// blocks of kStagedRows rows allow: the staging reads 8 n bytes per block,
// which counts as much as the matrix itself (900K rows of 49 entries: 530 MB
// of entries, 1.84 GB of segments with one group; the L2 delivers the latter
// at 11-17 TB/s).
//
// Entries are stored per (block, wave, segment) in row order, one word of
// column within the segment, turn and slot within the block beside the value,
// and taken in steps of 64, one entry per lane.  A wave owns its rows, so a
// step adds to the sums in LDS without atomics: in turn t the lanes whose
// entry is the t-th of its slot in this step read, add and write (one or two
// turns as a rule).  A slot is one row's sum, or one of several between which
// a row with many entries per segment deals them out, so that their turns do
// not hold the block up.  A slot's entries are added in column order within a
// group, the slots and then the groups in order, so the result does not
// depend on timing.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "cg_device.h"
#include "staged_internal.h"

namespace cgmi {

namespace {

constexpr int kSW = kStagedWaves;
constexpr int kST = kSW * kWave;

// s + v x, the product rounded first.
__device__ __forceinline__ double staged_add(double s, double v, double x) {
#pragma clang fp contract(off)
    return s + (double)v * (double)x;
}

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

typedef double Piece __attribute__((ext_vector_type(2)));

// The thread's 16-byte pieces of segment `seg` of p (the last segment again
// past the end).  As many loads are issued whichever segment it is, so that
// the compiler's count of loads in flight stays exact and a wait for older
// loads leaves these in flight.  The last segment's pieces are clamped to the
// vector's last whole one; what lies past it is stored by segment_store from
// `tail`.
template <int CH>
__device__ __forceinline__ void segment_load(const StagedDev &D, const double *__restrict__ p, int seg,
                                             Piece (&r)[CH]) {
    constexpr int E = 16 / sizeof(double);
    const double *const base = p + (int64_t)min(seg, D.nseg - 1) * D.seg_cols;   // uniform
    if (seg < D.nseg - 1 && D.seg_cols == CH * kST * E) {
#pragma unroll
        for (int u = 0; u < CH; ++u) __builtin_memcpy(&r[u], base + u * kST * E + (uint32_t)threadIdx.x * E, 16);
    } else {
        const int last = staged_last_pair(D.ncols - min(seg, D.nseg - 1) * D.seg_cols, D.seg_cols);
#pragma unroll
        for (int u = 0; u < CH; ++u)
            __builtin_memcpy(&r[u], base + (uint32_t)min((u * kST + (int)threadIdx.x) * E, last), 16);
    }
}

template <int CH>
__device__ __forceinline__ void segment_store(const StagedDev &D, int seg, double *buf,
                                              const Piece (&r)[CH], double tail) {
    constexpr int E = 16 / sizeof(double);
    Piece *const at = reinterpret_cast<Piece *>(buf) + threadIdx.x;
    const int pieces = D.seg_cols / E;
    if (pieces == CH * kST) {
#pragma unroll
        for (int u = 0; u < CH; ++u) at[u * kST] = r[u];
    } else {
#pragma unroll
        for (int u = 0; u < CH; ++u)
            if (u * kST + (int)threadIdx.x < pieces) at[u * kST] = r[u];
    }
    if (seg == D.nseg - 1) {   // the columns after the last whole piece
        __syncthreads();       // another thread's clamped piece covers them
        const int c = D.ncols / E * E + (int)threadIdx.x;
        if (c < D.ncols) buf[c - seg * D.seg_cols] = tail;
    }
}

// The first K steps of a list, [beg, end) of the entry arrays (which are
// padded so that these loads stay inside them).
template <int K>
struct Steps {
    int beg, end;
    uint32_t ix[K];
    double v[K];
    __device__ __forceinline__ void load(const uint32_t *__restrict__ idx, const double *__restrict__ val, int2 list) {
        const uint32_t lane = threadIdx.x & (kWave - 1);
        beg = list.x;
        end = list.y;
        const uint32_t *const ip = idx + beg;   // uniform
        const double *const vp = val + beg;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            ix[k] = ip[k * kWave + lane];
            v[k] = vp[k * kWave + lane];
        }
    }
};

// One step: the lanes that are on add v x to their slots, turn by turn.
__device__ __forceinline__ void staged_turns(bool on, uint32_t ix, double v, double x, double *y) {
    const int turn = on ? (int)staged_turn(ix) : -1;
    for (int t = 0;; ++t) {
        if (turn == t) {
            double &s = y[staged_slot(ix)];
            s = staged_add(s, v, x);
        }
        wave_sync();   // another lane may read this sum in the next turn or step
        if (!__any(turn > t)) break;
    }
}

template <int K>
__device__ __forceinline__ void staged_compute(const uint32_t *__restrict__ idx, const double *__restrict__ val,
                                               const Steps<K> &S, const double *buf, double *y) {
    const int lane = threadIdx.x & (kWave - 1);
    const int cnt = S.end - S.beg;
    double x[K];
#pragma unroll
    for (int k = 0; k < K; ++k) x[k] = buf[staged_col(S.ix[k])];   // past the list: another's column
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (k * kWave < cnt) staged_turns(k * kWave + lane < cnt, S.ix[k], S.v[k], x[k], y);
    for (int i = K * kWave; i < cnt; i += kWave) {
        const uint32_t ix = idx[S.beg + i + lane];   // past the last list: the arrays' padding
        const double v = val[S.beg + i + lane];
        staged_turns(i + lane < cnt, ix, v, buf[staged_col(ix)], y);
    }
}

// The sums of block blockIdx.x / ngroups over segment group blockIdx.x %
// ngroups, into D.part.
template <int CH, int K>
__global__ __launch_bounds__(kST) void k_staged_sums(StagedDev D, const double *__restrict__ p,
                                                     const int32_t *__restrict__ off,
                                                     const uint32_t *__restrict__ idx, const double *__restrict__ val,
                                                     const DevState *__restrict__ st) {
    extern __shared__ char lds_raw[];
    if (st && st->done) return;
    double *const buf0 = reinterpret_cast<double *>(lds_raw), *const buf1 = buf0 + D.seg_cols;
    double *const y = reinterpret_cast<double *>(buf1 + D.seg_cols);
    const int b = blockIdx.x / D.ngroups, g = blockIdx.x - b * D.ngroups;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x & (kWave - 1);
    for (int i = threadIdx.x, n = D.nslots[b]; i <= n; i += kST) y[i] = 0.0;   // and the dummy
    constexpr int E = 16 / sizeof(double);
    const int first = (int)((int64_t)D.nseg * g / D.ngroups), last = (int)((int64_t)D.nseg * (g + 1) / D.ngroups);
    const int list0 = (b * kSW + w) * D.nseg;
    // bounds of the wave's lists: 64 segments' in two registers, one segment
    // per lane, renewed every 62 (a list's bounds are read two segments ahead);
    // one by one as scalar loads they cost each segment a trip to memory
    int seg0 = 0, vbeg, vend;
    auto renew = [&](int s) {
        seg0 = s;
        const int l = list0 + min(s + lane, last - 1);
        vbeg = off[l];
        vend = off[l + 1];
    };
    auto bounds = [&](int s) {
        return make_int2(__builtin_amdgcn_readlane(vbeg, s - seg0), __builtin_amdgcn_readlane(vend, s - seg0));
    };
    renew(first);
    const int tail_col = D.ncols / E * E + (int)threadIdx.x;
    const double tail = tail_col < D.ncols ? p[tail_col] : 0.0;
    Piece P[CH];
    Steps<K> E0, E1;
    segment_load<CH>(D, p, first, P);
    segment_store<CH>(D, first, buf0, P, tail);
    E0.load(idx, val, bounds(first));
    segment_load<CH>(D, p, first + 1, P);
    int2 next = bounds(first + 1);
    __syncthreads();
    // segment s: the next list's entries are issued, this one's used, then
    // segment s + 1 goes from registers to the other buffer, which every wave
    // has finished reading at the barrier before, and s + 2 is issued
    auto step = [&](int s, const Steps<K> &cur, Steps<K> &nxt, const double *now, double *other) {
        nxt.load(idx, val, next);
        next = bounds(s + 2);
        staged_compute<K>(idx, val, cur, now, y);
        if (s + 1 < last) segment_store<CH>(D, s + 1, other, P, tail);
        segment_load<CH>(D, p, s + 2, P);
        __syncthreads();
    };
    for (int s = first; s < last; s += 2) {
        if (s - seg0 == kWave - 2) renew(s);
        step(s, E0, E1, buf0, buf1);
        if (s + 1 < last) step(s + 1, E1, E0, buf1, buf0);
    }
    double *const part = D.part + (int64_t)g * D.m;
    const int row0 = D.row0[b * kSW], r0 = D.row0[b * kSW + w], r1 = D.row0[b * kSW + w + 1];
    for (int r = r0 + lane; r < r1; r += kWave) {
        const uint32_t u = D.slots ? D.slots[r] : (uint32_t)(r - row0) | 1u << 16;
        double s = y[u & 0xFFFFu];
        for (uint32_t i = 1; i < u >> 16; ++i) s += y[(u & 0xFFFFu) + i];
        part[r] = s;
    }
}

// The end of every mode of k_spmv on the groups' sums; one partial per
// workgroup.
template <int MODE>
__global__ __launch_bounds__(kBlock) void k_staged_end(int32_t m, int32_t ngroups, const double *__restrict__ part,
                                                       SpmvArgs<double> a, double *__restrict__ out, Partials in0,
                                                       Partials in1, DevState *__restrict__ st, int flags) {
    __shared__ double sh[kWavesPerBlock];
    __shared__ double bc;
    if (flags & kFlagCheckDone) {
        if (st->done) return;
        if (flags & kFlagFirstIter) {
            // stop test at the top of iteration 0 from the setup partials
            const double rr = reduce_partials(in0, sh, &bc);
            const double bb = reduce_partials(in1, sh, &bc);
            const bool conv = stop_test(rr, bb, st->tol);
            const bool stop = conv || st->maxit <= 0;
            if (is_block0_thread0()) {
                st->rho[0] = rr;
                st->rr = rr;
                st->bb = bb;
                if (stop) st->done = conv ? kDoneConverged : kDoneMaxit;
            }
            if (stop) return;
        }
    }
    double acc0 = 0.0, acc1 = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < m; i += (int64_t)gridDim.x * kBlock) {
        double s = part[i];
        for (int g = 1; g < ngroups; ++g) s += part[(int64_t)g * m + i];
        emit_row<MODE, double>(a, (int)i, s, acc0, acc1);
    }
    if (MODE == kSpmvPlain) return;
    const double s0 = block_sum<kBlock>(acc0, sh);
    double s1 = 0.0;
    if (MODE == kSpmvResidual) s1 = block_sum<kBlock>(acc1, sh);
    if (threadIdx.x == 0) {
        out[blockIdx.x] = s0;
        if (MODE == kSpmvResidual) out[gridDim.x + blockIdx.x] = s1;
    }
}

hipError_t launch_sums(const StagedDev &D, const double *p, const DevState *st, hipStream_t s) {
    const size_t lds = staged_lds(D.seg_cols, D.max_slots);
    const int chunks = (int)((D.seg_cols * sizeof(double) / 16 + kST - 1) / kST);
    if (lds > kStagedLds || chunks > kStagedChunks || D.ncols - (D.nseg - 1) * D.seg_cols < 2)
        return hipErrorInvalidValue;
#define CGMI_STAGED(CH, K)                                                                                    \
    hipLaunchKernelGGL((k_staged_sums<CH, K>), dim3(D.nblocks * D.ngroups), dim3(kST), lds, s, D, p, D.off, \
                       D.idx, D.val, st)
    // as many steps ahead as a list has at the most on average: a step costs
    // its instructions also where the list has ended (900K rows of 49 entries,
    // 2.6 steps a list: 211 us with 6, 170 with 3, 182 with 2; 700K of 41: 150,
    // 122 and 128)
    const int K = std::min(std::max(D.ahead, 2), kStagedAhead);
    if (chunks <= 3) {
        if (K == 2) CGMI_STAGED(3, 2);
        else if (K == 3) CGMI_STAGED(3, 3);
        else if (K == 4) CGMI_STAGED(3, 4);
        else if (K == 5) CGMI_STAGED(3, 5);
        else CGMI_STAGED(3, kStagedAhead);
    } else {
        if (K == 2) CGMI_STAGED(4, 2);
        else if (K == 3) CGMI_STAGED(4, 3);
        else if (K == 4) CGMI_STAGED(4, 4);
        else if (K == 5) CGMI_STAGED(4, 5);
        else CGMI_STAGED(4, kStagedAhead);
    }
#undef CGMI_STAGED
    return hipGetLastError();
}

template <int MODE>
hipError_t launch_mode(const StagedDev &D, int grid, const SpmvArgs<double> &a, double *out, Partials in0,
                       Partials in1, DevState *st, int flags, hipStream_t s) {
    const hipError_t e = launch_sums(D, a.p, st, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_staged_end<MODE>), dim3(grid), dim3(kBlock), 0, s, D.m, D.ngroups, D.part, a, out, in0,
                       in1, st, flags);
    return hipGetLastError();
}

hipError_t allow_lds() {
    hipError_t e = hipSuccess;
    for (const void *fn : {reinterpret_cast<const void *>(k_staged_sums<3, 2>),
                           reinterpret_cast<const void *>(k_staged_sums<4, 2>),
                           reinterpret_cast<const void *>(k_staged_sums<3, 3>),
                           reinterpret_cast<const void *>(k_staged_sums<3, 4>),
                           reinterpret_cast<const void *>(k_staged_sums<3, 5>),
                           reinterpret_cast<const void *>(k_staged_sums<3, kStagedAhead>),
                           reinterpret_cast<const void *>(k_staged_sums<4, 3>),
                           reinterpret_cast<const void *>(k_staged_sums<4, 4>),
                           reinterpret_cast<const void *>(k_staged_sums<4, 5>),
                           reinterpret_cast<const void *>(k_staged_sums<4, kStagedAhead>)})
        if (e == hipSuccess) e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kStagedLds);
    return e;
}

}  // namespace

hipError_t staged_setup() {
    return allow_lds();
}

hipError_t launch_spmv_staged(const StagedDev &D, int grid, const double *p, double *q, const double *p_own,
                              const double *b, double *p_dst, double *out, Partials in0, Partials in1,
                              DevState *st, int mode, int k0_check, hipStream_t s) {
    const SpmvArgs<double> a{p, q, p_own, b, p_dst};
    const int flags = st ? kFlagCheckDone | (mode == kSpmvDot && k0_check ? kFlagFirstIter : 0) : 0;
    switch (mode) {
        case kSpmvPlain: return launch_mode<kSpmvPlain>(D, grid, a, out, in0, in1, st, flags, s);
        case kSpmvDot: return launch_mode<kSpmvDot>(D, grid, a, out, in0, in1, st, flags, s);
        case kSpmvResidual: return launch_mode<kSpmvResidual>(D, grid, a, out, in0, in1, nullptr, 0, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace cgmi
