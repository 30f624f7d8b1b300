// kernels_batch.hip -- batched multi-RHS CG in one persistent launch (gfx950).
//
// Each pair (system k, right-hand side j) runs the CG recurrence of
// Algorithm 1 with its own scalars.  A team of workgroups owns the rows of
// system k for the whole launch; a row takes as many lanes (a power of two) as
// its right-hand sides need, so the values of one row of a vector are
// contiguous (16 right-hand sides: a 128-byte line, which a gathered p_c of
// all of them is too) and few lanes idle (always 16 lanes: 511K rows with one
// right-hand side 135 us per iteration, now 30; with 5, 138 and 76).
//
// A workgroup works through a list of items, each a (system, rank in its
// team) pair, one after the other: heavy systems get teams of their own,
// while light systems that a single workgroup solves are packed, several to
// a workgroup, so that the grid's work evens out.  The host builds the lists
// (first-fit decreasing on weights n_k^e); an item that belongs to a team of
// more than one workgroup is always its workgroup's only item, so no team
// barrier waits on a workgroup that is still busy with an earlier system.
//
// One iteration is three phases separated by team barriers:
//   A: q = A p on the team's rows, partial p^T q per right-hand side;
//   B: alpha = rho / p^T q (team sum), r -= alpha q, partial r^T r;
//   C: stop test and beta = r^T r / rho (team sum), x += alpha p for every
//      right-hand side updated in B, p = r + beta p for those still running.
// Algorithm 1 updates x with r; x is not read again before C, which reads
// the same p, so the x update is done there and B does not read p.
// Every workgroup of a team sums the team's partials itself in a fixed order,
// so all of them take identical decisions (and results are reproducible for
// a fixed schedule).  Of the three barriers only the one after C has to move
// vectors between workgroups (the p that A gathers); the other two exchange
// partial sums alone, in words that carry their own validity (publish), and
// leave every cache as it is.  With a cache write-back and invalidation by
// every wave at all three, and 256 threads to a workgroup, an iteration of 24
// diffusion systems of side 32-256 with 16 right-hand sides took 607 us, 330 of
// them in the barriers; so, and with 1024 threads, it took 181 us.  Waits are
// bounded by a wall-clock limit; on expiry the error flag ends every team.
#include <hip/hip_runtime.h>
#include <math.h>

#include <type_traits>

#include "batch_internal.h"

namespace cgmi {

namespace {

constexpr int kL = kBatchLanes;
constexpr int kStripSteps = 4;   // steps a line has at least where phase A goes by strips
enum { kSlotPQ = 0, kSlotRR = 1, kSlotBB = 2, kSlotTrue = 3 };
enum { kStOk = 0, kStMaxit = 1, kStBreakdown = -4 };

template <int NT>
struct Shared {
    double red[NT / 64][kL];
    double tmp[NT];
    double sum[kL];
    double rho[kL], bb[kL], alpha[kL], beta[kL], rr_last[kL];
    int active[kL], status[kL], iter[kL], zero_b[kL];
    int upd[kL];   // updated r (and owes the x update) in this iteration's phase B
    int any, any_upd;
    int ok;
};

// The value of the lane N further on in its row of 16.
template <int N>
__device__ __forceinline__ double row_rotate(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x120 + N, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x120 + N, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

// Sum over the workgroup for each right-hand side: a lane holds V consecutive
// right-hand sides j0 .. j0+V-1 (acc[v] for j0 + v); lanes with the same j0
// are `lanes` apart.  The sums are returned to threads 0 .. 15.
template <int NT, int V>
__device__ __forceinline__ double wg_partial(const double (&acc)[V], int lanes, Shared<NT> &S) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    double v[V];
#pragma unroll
    for (int q = 0; q < V; ++q) {
        v[q] = acc[q];
        v[q] += __shfl_xor(v[q], 32, 64);
        v[q] += __shfl_xor(v[q], 16, 64);
        // within the rows of 16 lanes: what has the period 2 o already, a
        // rotation by o pairs like an exchange
        if (lanes <= 8) v[q] += row_rotate<8>(v[q]);
        if (lanes <= 4) v[q] += row_rotate<4>(v[q]);
        if (lanes <= 2) v[q] += row_rotate<2>(v[q]);
        if (lanes <= 1) v[q] += row_rotate<1>(v[q]);
    }
    if (lane < lanes)
#pragma unroll
        for (int q = 0; q < V; ++q) S.red[wv][lane * V + q] = v[q];
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x < kL) {
        s = S.red[0][threadIdx.x];
#pragma unroll
        for (int q = 1; q < NT / 64; ++q) s += S.red[q][threadIdx.x];
    }
    return s;
}

// One step of a bounded wait: false when the launch is being abandoned (the
// error flag is set, or the wait that began at t0 exceeds its limit).
__device__ __forceinline__ bool wait_on(const BatchArgs &a, uint64_t t0) {
    if (__hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return false;
    if ((int64_t)(wall_clock64() - t0) > a.timeout_ticks) {
        __hip_atomic_store(a.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return false;
    }
    __builtin_amdgcn_s_sleep(1);
    return true;
}

__device__ __forceinline__ uint64_t *part_words(const BatchArgs &a, int wg, int slot) {
    return a.part + ((int64_t)wg * kBatchSlots + slot) * 2 * kL;
}

// Publishes the workgroup's sums of a slot (value v of threads 0 .. 15) for
// the team, tagged with the episode (> 0, higher in every use of the slot):
// two relaxed 64-bit words, each half of the value's bits beside the tag.  A
// reader takes a word for the episode it waits for only with that tag, so
// neither side needs an ordering between different words: no fence, no
// counter, one trip through memory instead of two.
__device__ __forceinline__ void publish(const BatchArgs &a, int slot, int episode, double v) {
    if (threadIdx.x >= kL) return;
    uint64_t *const w = part_words(a, blockIdx.x, slot) + threadIdx.x;
    const uint64_t bits = (uint64_t)__double_as_longlong(v), tag = (uint64_t)(uint32_t)episode << 32;
    __hip_atomic_store(w, tag | (bits & 0xFFFFFFFFu), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(w + kL, tag | bits >> 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Team sum of one slot for every j, in a fixed order, into S.sum: waits for
// the words of every member (first .. first + T - 1) with the episode's tag.
// A slot is written again only after its writer has seen every member's words
// of a later episode of another slot, hence after every member has read it.
// False when the launch is being abandoned.
template <int NT>
__device__ __forceinline__ bool team_sum(const BatchArgs &a, int first, int T, int slot, int episode, double mine,
                                         Shared<NT> &S) {
    if (T == 1) {
        if (threadIdx.x < kL) S.sum[threadIdx.x] = mine;
        __syncthreads();
        return true;
    }
    publish(a, slot, episode, mine);
    const int j = threadIdx.x & (kL - 1), g = threadIdx.x / kL;
    double v = 0.0;
    bool ok = true;
    if (g < T) {
        const uint64_t t0 = wall_clock64();
        for (int r = g; r < T && ok; r += NT / kL) {
            const uint64_t *const w = part_words(a, first + r, slot) + j;
            uint64_t lo, hi;
            for (;;) {
                lo = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                hi = __hip_atomic_load(w + kL, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if ((uint32_t)(lo >> 32) == (uint32_t)episode && (uint32_t)(hi >> 32) == (uint32_t)episode) break;
                if (!wait_on(a, t0)) {
                    ok = false;
                    break;
                }
            }
            v += __longlong_as_double((long long)(hi << 32 | (lo & 0xFFFFFFFFu)));
        }
    }
    if (!ok) S.ok = 0;
    S.tmp[threadIdx.x] = v;
    __syncthreads();
    if (threadIdx.x < kL) {
        double s = 0.0;
        const int groups = min(T, NT / kL);
        for (int q = 0; q < groups; ++q) s += S.tmp[q * kL + threadIdx.x];
        S.sum[threadIdx.x] = s;
    }
    __syncthreads();
    return S.ok != 0;
}

// Barrier of a team (T workgroups) that makes the vectors its members wrote
// visible to all of them.  Returns false when the launch is being abandoned.
//
// Team members sit on different XCDs, whose L2 caches are not coherent with
// each other: what a member wrote has to leave its XCD's L2 before another
// reads it, and the reader's XCD has to drop what it holds of it.  Both act on
// a whole L2, so one wave of each workgroup does them for the workgroup; their
// cost grows with the number of waves that do (every wave of 768 workgroups
// of 4: 111 us per barrier).  Every wave waits until its stores have reached
// the L2 (the wait is spelled out: a workgroup barrier alone orders the waves
// of a workgroup, which share a CU's L1, and need not wait for the L2), the
// workgroup synchronises, and wave 0's agent-scope release fence writes the L2
// back before its first thread marks the episode in the workgroup's word.  The
// waves that wait for the members' words then issue the agent-scope acquire
// fence, wait for it, and the second workgroup barrier lets the others read
// through the L1 and L2 they have invalidated.
template <int NT>
__device__ __forceinline__ bool team_sync(const BatchArgs &a, int first, int T, int episode, Shared<NT> &S) {
    if (T == 1) {
        __syncthreads();
        return true;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x < 64) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        if (threadIdx.x == 0)
            __hip_atomic_store(a.sync + blockIdx.x, episode, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if ((int)(threadIdx.x & ~63u) < T) {   // the waves with a member to wait for
        bool ok = true;
        const uint64_t t0 = wall_clock64();
        for (int r = threadIdx.x; r < T && ok; r += NT)
            while (__hip_atomic_load(a.sync + first + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < episode)
                if (!wait_on(a, t0)) {
                    ok = false;
                    break;
                }
        if (!ok) S.ok = 0;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    __syncthreads();
    return S.ok != 0;
}

__device__ __forceinline__ bool stop_test(double rr, double bb, double tol) {
    return sqrt(rr) < tol * sqrt(bb) || rr == 0.0;
}

// V consecutive float64 values at p[idx] (16-byte aligned when V = 2).
template <int V>
__device__ __forceinline__ void ldv(const double *__restrict__ p, int64_t idx, double (&o)[V]) {
    if constexpr (V == 2) {
        const double2 t = *reinterpret_cast<const double2 *>(p + idx);
        o[0] = t.x;
        o[1] = t.y;
    } else {
        o[0] = p[idx];
    }
}
template <int V>
__device__ __forceinline__ void stv(double *__restrict__ p, int64_t idx, const double (&v)[V]) {
    if constexpr (V == 2) {
        *reinterpret_cast<double2 *>(p + idx) = double2{v[0], v[1]};
    } else {
        p[idx] = v[0];
    }
}

// What a workgroup keeps in LDS of the vectors that no other workgroup reads
// (511K rows with 16 right-hand sides, 2000 rows of which 1152 fit: 181 to 161
// us per iteration): r of its first nr rows, q of its first nq and x of its first nx (nx <= nq <=
// nr; r is touched three times an iteration, the others twice).  All three are
// read and written by the same thread of a row, but q, which phase A writes.
template <bool ON>
struct Keep {
    double *r, *q, *x;
    int nr, nq, nx;
    template <int V>
    __device__ __forceinline__ void put(double *kept, int rows, double *__restrict__ v, int64_t local, int64_t idx,
                                        int nrhs, int j0, const double (&s)[V]) const {
        if (ON && local < rows) stv<V>(kept, (int)local * nrhs + j0, s);
        else stv<V>(v, idx, s);
    }
};

// sum_k val[k] * v[col[k] * nr + j0 + q] for one row and the lane's V
// right-hand sides, in CSR order, each product and sum rounded separately (as
// the oracle's SpMV).  Rows of up to kShort entries load all their columns
// and values first (clamped indices, all independent), then issue all
// gathers, so a row costs two memory round trips instead of one per entry;
// longer rows take a plain loop.
constexpr int kShort = 8;

template <int V>
__device__ __forceinline__ void row_dot(const BatchArgs &a, int64_t row, const double *__restrict__ v,
                                        int nr, int j0, double (&s)[V]) {
#pragma clang fp contract(off)
    const int k0 = a.rp[row], k1 = a.rp[row + 1];
    const int len = k1 - k0;
#pragma unroll
    for (int q = 0; q < V; ++q) s[q] = 0.0;
    if (len <= 0) return;
    if (len <= kShort) {
        int c[kShort];
        double w[kShort], pv[kShort][V];
#pragma unroll
        for (int e = 0; e < kShort; ++e) {
            const int k = k0 + (e < len ? e : 0);
            c[e] = a.ci[k];
            w[e] = a.val[k];
        }
#pragma unroll
        for (int e = 0; e < kShort; ++e) ldv<V>(v, (int64_t)c[e] * nr + j0, pv[e]);
#pragma unroll
        for (int e = 0; e < kShort; ++e)
            if (e < len)
#pragma unroll
                for (int q = 0; q < V; ++q) s[q] += w[e] * pv[e][q];
        return;
    }
    for (int k = k0; k < k1; ++k) {
        double pv[V];
        ldv<V>(v, (int64_t)a.ci[k] * nr + j0, pv);
#pragma unroll
        for (int q = 0; q < V; ++q) s[q] += a.val[k] * pv[q];
    }
}

// Columns and values of a row of at most kPipe entries (clamped: entries
// past the row repeat its first, an empty row reads entry 0).  kPipe is 5 for a
// batch of rows of at most 5 entries, else 6: every entry more is two loads and
// a gather per row, needed or not (24 diffusion systems, 16 right-hand sides:
// 148 us per iteration with 5, 161 with 6).
template <int kPipe>
__device__ __forceinline__ void row_cw(const BatchArgs &a, int k0, int len, int (&c)[kPipe],
                                       double (&w)[kPipe]) {
    const int base = len > 0 ? k0 : 0;
#pragma unroll
    for (int e = 0; e < kPipe; ++e) {
        const int k = base + (e < len ? e : 0);
        c[e] = a.ci[k];
        w[e] = a.val[k];
    }
}

// Phase A over the thread's rows lo + rsub, lo + rsub + RS, ...: q = A p and
// the partial p^T q, with three rows in flight (while the current row's
// gathers return, the next row's columns and values and the row pointers of
// the one after are loading), so a row costs about one memory round trip
// instead of three.  Sums as row_dot: CSR order, each product and sum
// rounded; rows longer than kPipe go entry by entry in the same order.
template <int V, int kPipe, class K_>
__device__ __forceinline__ void spmv_rows_pipelined(const BatchArgs &a, const K_ &K, int64_t lo, int64_t hi, int RS,
                                                    int rsub, int nr, int j0, const bool (&on)[V],
                                                    double (&acc)[V]) {
#pragma clang fp contract(off)
    int64_t row = lo + rsub;
    if (row >= hi) return;
    int k0c = a.rp[row], lenc = a.rp[row + 1] - k0c;
    int cc[kPipe];
    double wc[kPipe];
    row_cw<kPipe>(a, k0c, lenc, cc, wc);
    int k0n = 0, k1n = 0;
    if (row + RS < hi) {
        k0n = a.rp[row + RS];
        k1n = a.rp[row + RS + 1];
    }
    for (; row < hi; row += RS) {
        double pv[kPipe][V], po[V];
#pragma unroll
        for (int e = 0; e < kPipe; ++e) ldv<V>(a.P, (int64_t)cc[e] * nr + j0, pv[e]);
        const int64_t idx = row * nr + j0;
        ldv<V>(a.P, idx, po);
        int cn[kPipe];
        double wn[kPipe];
        row_cw<kPipe>(a, k0n, k1n - k0n, cn, wn);
        int k0nn = 0, k1nn = 0;
        if (row + 2 * RS < hi) {
            k0nn = a.rp[row + 2 * RS];
            k1nn = a.rp[row + 2 * RS + 1];
        }
        double sv[V];
#pragma unroll
        for (int q = 0; q < V; ++q) sv[q] = 0.0;
        if (lenc <= kPipe) {
#pragma unroll
            for (int e = 0; e < kPipe; ++e)
                if (e < lenc)
#pragma unroll
                    for (int q = 0; q < V; ++q) sv[q] += wc[e] * pv[e][q];
        } else {
            for (int k = k0c; k < k0c + lenc; ++k) {
                double g[V];
                ldv<V>(a.P, (int64_t)a.ci[k] * nr + j0, g);
                const double wk = a.val[k];
#pragma unroll
                for (int q = 0; q < V; ++q) sv[q] += wk * g[q];
            }
        }
        K.template put<V>(K.q, K.nq, a.Q, row - lo, idx, nr, j0, sv);
#pragma unroll
        for (int q = 0; q < V; ++q)
            if (on[q]) acc[q] = fma(po[q], sv[q], acc[q]);
        k0c = k0n;
        lenc = k1n - k0n;
#pragma unroll
        for (int e = 0; e < kPipe; ++e) {
            cc[e] = cn[e];
            wc[e] = wn[e];
        }
        k0n = k0nn;
        k1n = k1nn;
    }
}

// Phase A in strip order, for systems whose rows form lines of D rows (a
// grid numbered line by line; the host sets D where every column offset is
// either below D/4 or within D/4 of D): the workgroup's rows are visited as
// columns x in [s RS, (s+1) RS) of the lines, strip s after strip s - 1,
// each strip walked down the workgroup's lines.  A row's neighbours in the
// lines above and below are then used within a few steps of each other, so
// the gathered lines of p stay in the L2 of every workgroup at once (in row
// order each workgroup keeps two whole lines in flight, 128 KB at D = 512
// and 16 right-hand sides, more than an XCD's L2 holds for all its
// workgroups).  Rows are summed as in spmv_rows_pipelined, three in flight;
// only the order of the rows in the thread's partial p^T q changes.
template <int V, int kPipe, class K_>
__device__ __forceinline__ void spmv_rows_strips(const BatchArgs &a, const K_ &K, int64_t off, int64_t lo, int64_t hi, int D,
                                                 int RS, int rsub, int nr, int j0, const bool (&on)[V],
                                                 double (&acc)[V]) {
#pragma clang fp contract(off)
    const int64_t l0 = lo - off, l1 = hi - off;       // local rows [l0, l1)
    if (l1 <= l0) return;
    const int64_t y0 = l0 / D, nlines = (l1 - 1) / D - y0 + 1;
    const int nstrips = (D + RS - 1) / RS;
    const int64_t nsteps = nlines * nstrips;
    // global row of step t, or -1 (a column past the line, or outside [lo, hi))
    auto row_at = [&](int64_t t) -> int64_t {
        if (t >= nsteps) return -1;
        const int64_t strip = t / nlines;
        const int64_t x = strip * RS + rsub;
        const int64_t r = (y0 + (t - strip * nlines)) * D + x;
        return (x < D && r >= l0 && r < l1) ? off + r : -1;
    };
    int64_t row = row_at(0);
    int k0c = 0, lenc = 0;
    if (row >= 0) {
        k0c = a.rp[row];
        lenc = a.rp[row + 1] - k0c;
    }
    int cc[kPipe];
    double wc[kPipe];
    row_cw<kPipe>(a, k0c, lenc, cc, wc);
    int64_t rown = row_at(1);
    int k0n = 0, k1n = 0;
    if (rown >= 0) {
        k0n = a.rp[rown];
        k1n = a.rp[rown + 1];
    }
    for (int64_t t = 0; t < nsteps; ++t) {
        double pv[kPipe][V], po[V];
#pragma unroll
        for (int e = 0; e < kPipe; ++e) ldv<V>(a.P, (int64_t)cc[e] * nr + j0, pv[e]);
        const int64_t idx = (row >= 0 ? row : lo) * nr + j0;
        ldv<V>(a.P, idx, po);
        int cn[kPipe];
        double wn[kPipe];
        row_cw<kPipe>(a, k0n, k1n - k0n, cn, wn);
        const int64_t rownn = row_at(t + 2);
        int k0nn = 0, k1nn = 0;
        if (rownn >= 0) {
            k0nn = a.rp[rownn];
            k1nn = a.rp[rownn + 1];
        }
        double sv[V];
#pragma unroll
        for (int q = 0; q < V; ++q) sv[q] = 0.0;
        if (lenc <= kPipe) {
#pragma unroll
            for (int e = 0; e < kPipe; ++e)
                if (e < lenc)
#pragma unroll
                    for (int q = 0; q < V; ++q) sv[q] += wc[e] * pv[e][q];
        } else {
            for (int k = k0c; k < k0c + lenc; ++k) {
                double g[V];
                ldv<V>(a.P, (int64_t)a.ci[k] * nr + j0, g);
                const double wk = a.val[k];
#pragma unroll
                for (int q = 0; q < V; ++q) sv[q] += wk * g[q];
            }
        }
        if (row >= 0) {
            K.template put<V>(K.q, K.nq, a.Q, row - lo, idx, nr, j0, sv);
#pragma unroll
            for (int q = 0; q < V; ++q)
                if (on[q]) acc[q] = fma(po[q], sv[q], acc[q]);
        }
        row = rown;
        rown = rownn;
        k0c = k0n;
        lenc = k1n - k0n;
#pragma unroll
        for (int e = 0; e < kPipe; ++e) {
            cc[e] = cn[e];
            wc[e] = wn[e];
        }
        k0n = k0nn;
        k1n = k1nn;
    }
}

extern __shared__ double s_keep[];   // [a.keep]

// U: rows a thread advances per step in the setup and the vector phases B
// and C (phase A keeps three rows in flight by itself); V: right-hand sides
// per lane (2 needs an even nrhs and 16-byte aligned vectors).
// One system's solve by this workgroup as member `rank` of its team (the
// whole solve when the team is the workgroup alone).  False when the launch
// is being abandoned (a team wait gave up).
template <int NT, int U, int V, int E>
__device__ __forceinline__ bool batch_solve_one(const BatchArgs &a, int sys, int rank, Shared<NT> &S) {
    const int lanes = 1 << a.lane_bits;  // lanes per row
    const int RS = NT >> a.lane_bits;    // rows per workgroup step
    const int T = a.team_size[sys], first = a.team_first[sys];
    const int64_t off = a.row_off[sys], n = a.row_off[sys + 1] - off;
    const int64_t lo = off + n * rank / T, hi = off + n * (rank + 1) / T;
    const int nr = a.nrhs;
    const int j0 = (threadIdx.x & (lanes - 1)) * V, rsub = threadIdx.x >> a.lane_bits;
    const bool lane_on = j0 < nr;
    int episode = 1;
    constexpr bool kept = NT == 1024;   // else none is (batch_keep)
    Keep<kept> K{};
    if (kept) {
        // whole steps, or all rows
        const int rows = (int)min(hi - lo, (int64_t)(1 << 30)), most = a.keep / nr;
        auto part = [&](int room) { return room >= rows ? rows : max(room, 0) / RS * RS; };
        K.nr = part(most);
        K.nq = min(part(most - K.nr), K.nr);
        K.nx = min(part(most - K.nr - K.nq), K.nq);
        K.r = s_keep;
        K.q = K.r + (int64_t)K.nr * nr;
        K.x = K.q + (int64_t)K.nq * nr;
    }
    // f(kept in LDS: r, second) over the thread's rows, U a step, in order:
    // those with r and the second vector (q or x) there, with r alone, neither
    auto for_rows = [&](int second, auto f) {
        auto run = [&](int from, int to, auto kept_r, auto kept_s) {
            for (int64_t r0 = lo + from; r0 < lo + to; r0 += RS * U)
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int64_t row = r0 + u * RS + rsub;
                    if (row < lo + to) f(row, kept_r, kept_s);
                }
        };
        if (kept) {
            run(0, second, std::true_type{}, std::true_type{});
            run(second, K.nr, std::true_type{}, std::false_type{});
        }
        run(K.nr, (int)(hi - lo), std::false_type{}, std::false_type{});
    };

    // setup: r = b - A x, p = r; partial r^T r and b^T b
    {
        double arr[V], abb[V];
#pragma unroll
        for (int q = 0; q < V; ++q) arr[q] = abb[q] = 0.0;
        if (lane_on)
            for (int64_t r0 = lo; r0 < hi; r0 += RS * U)
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int64_t row = r0 + u * RS + rsub;
                    if (row < hi) {
                        double s[V], bv[V], rv[V];
                        row_dot<V>(a, row, a.X, nr, j0, s);
                        const int64_t idx = row * nr + j0;
                        ldv<V>(a.B, idx, bv);
#pragma unroll
                        for (int q = 0; q < V; ++q) {
                            rv[q] = bv[q] - s[q];
                            arr[q] = fma(rv[q], rv[q], arr[q]);
                            abb[q] = fma(bv[q], bv[q], abb[q]);
                        }
                        K.template put<V>(K.r, K.nr, a.R, row - lo, idx, nr, j0, rv);
                        stv<V>(a.P, idx, rv);
                        if (kept && row - lo < K.nx) {
                            double xv[V];
                            ldv<V>(a.X, idx, xv);
                            stv<V>(K.x, (row - lo) * nr + j0, xv);
                        }
                    }
                }
        const double rr = wg_partial<NT, V>(arr, lanes, S);
        if (!team_sync<NT>(a, first, T, episode, S)) return false;
        if (!team_sum<NT>(a, first, T, kSlotRR, episode, rr, S)) return false;
        if (threadIdx.x < kL) S.rr_last[threadIdx.x] = S.sum[threadIdx.x];
        const double bb = wg_partial<NT, V>(abb, lanes, S);
        if (!team_sum<NT>(a, first, T, kSlotBB, episode, bb, S)) return false;
    }
    if (threadIdx.x < kL) {
        const int t = threadIdx.x;
        const double rr = S.rr_last[t], bb = S.sum[t];
        S.rho[t] = rr;
        S.bb[t] = bb;
        S.iter[t] = 0;
        S.zero_b[t] = 0;
        S.active[t] = 0;
        S.status[t] = kStOk;
        if (t < nr) {
            if (bb == 0.0) S.zero_b[t] = 1;
            else if (stop_test(rr, bb, a.tol)) S.status[t] = kStOk;
            else if (a.maxit <= 0) S.status[t] = kStMaxit;
            else S.active[t] = 1;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int any = 0;
        for (int t = 0; t < kL; ++t) any |= S.active[t];
        S.any = any;
    }
    __syncthreads();

    for (int k = 0; S.any; ++k) {
        // A: q = A p, partial p^T q
        {
            bool on[V];
            bool any_on = false;
#pragma unroll
            for (int q = 0; q < V; ++q) {
                on[q] = lane_on && S.active[j0 + q];
                any_on |= on[q];
            }
            double acc[V];
#pragma unroll
            for (int q = 0; q < V; ++q) acc[q] = 0.0;
            if (any_on && lane_on) {
                // (strips only where a step is a small part of a line: the
                // last strip's lanes past the line idle)
                const int D = a.strip[sys];
                if (D >= kStripSteps * RS)
                    spmv_rows_strips<V, E>(a, K, off, lo, hi, D, RS, rsub, nr, j0, on, acc);
                else
                    spmv_rows_pipelined<V, E>(a, K, lo, hi, RS, rsub, nr, j0, on, acc);
            }
            const double pq = wg_partial<NT, V>(acc, lanes, S);
            if (!team_sum<NT>(a, first, T, kSlotPQ, ++episode, pq, S)) return false;
        }
        if (threadIdx.x < kL) {
            const int t = threadIdx.x;
            S.alpha[t] = 0.0;
            S.upd[t] = 0;
            if (S.active[t]) {
                const double pq = S.sum[t];
                if (!(pq > 0.0) || !isfinite(pq)) {
                    S.status[t] = kStBreakdown;
                    S.iter[t] = k;
                    S.active[t] = 0;
                } else {
                    S.alpha[t] = S.rho[t] / pq;
                    S.upd[t] = 1;
                }
            }
        }
        __syncthreads();
        // B: r -= alpha q, partial r^T r
        {
            bool on[V];
            bool any_on = false;
            double alpha[V], acc[V];
#pragma unroll
            for (int q = 0; q < V; ++q) {
                on[q] = lane_on && S.active[j0 + q];
                any_on |= on[q];
                alpha[q] = on[q] ? S.alpha[j0 + q] : 0.0;
                acc[q] = 0.0;
            }
            if (any_on)
                for_rows(K.nq, [&](int64_t row, auto kept_r, auto kept_q) {
                    const int64_t idx = row * nr + j0;
                    const int at = (int)(row - lo) * nr + j0;
                    double qv[V], rv[V];
                    if constexpr (decltype(kept_q)::value) ldv<V>(K.q, at, qv);
                    else ldv<V>(a.Q, idx, qv);
                    if constexpr (decltype(kept_r)::value) ldv<V>(K.r, at, rv);
                    else ldv<V>(a.R, idx, rv);
#pragma unroll
                    for (int q = 0; q < V; ++q) {
                        if (on[q]) {
                            rv[q] = fma(-alpha[q], qv[q], rv[q]);
                            acc[q] = fma(rv[q], rv[q], acc[q]);
                        }
                    }
                    if constexpr (decltype(kept_r)::value) stv<V>(K.r, at, rv);
                    else stv<V>(a.R, idx, rv);
                });
            const double rr = wg_partial<NT, V>(acc, lanes, S);
            if (!team_sum<NT>(a, first, T, kSlotRR, ++episode, rr, S)) return false;
        }
        if (threadIdx.x < kL) {
            const int t = threadIdx.x;
            S.beta[t] = 0.0;
            if (S.active[t]) {
                const double rr = S.sum[t];
                S.iter[t] = k + 1;
                S.rr_last[t] = rr;
                S.beta[t] = rr / S.rho[t];
                S.rho[t] = rr;
                if (stop_test(rr, S.bb[t], a.tol)) {
                    S.status[t] = kStOk;
                    S.active[t] = 0;
                } else if (k + 1 >= a.maxit) {
                    S.status[t] = kStMaxit;
                    S.active[t] = 0;
                }
            }
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            int any = 0, any_upd = 0;
            for (int t = 0; t < kL; ++t) {
                any |= S.active[t];
                any_upd |= S.upd[t];
            }
            S.any = any;
            S.any_upd = any_upd;
        }
        __syncthreads();
        if (!S.any_upd) break;   // every right-hand side broke down in A: nothing owed
        // C: x += alpha p (right-hand sides updated in B), p = r + beta p (still running)
        {
            bool on[V], up[V];
            bool any_on = false, any_up = false;
            double alpha[V], beta[V];
#pragma unroll
            for (int q = 0; q < V; ++q) {
                on[q] = lane_on && S.active[j0 + q];
                up[q] = lane_on && S.upd[j0 + q];
                any_on |= on[q];
                any_up |= up[q];
                alpha[q] = S.alpha[j0 + q];
                beta[q] = S.beta[j0 + q];
            }
            if (any_up)
                for_rows(K.nx, [&](int64_t row, auto kept_r, auto kept_x) {
                    const int64_t idx = row * nr + j0;
                    const int at = (int)(row - lo) * nr + j0;
                    double pv[V], xv[V], rv[V];
                    ldv<V>(a.P, idx, pv);
                    if constexpr (decltype(kept_x)::value) ldv<V>(K.x, at, xv);
                    else ldv<V>(a.X, idx, xv);
                    if (any_on) {
                        if constexpr (decltype(kept_r)::value) ldv<V>(K.r, at, rv);
                        else ldv<V>(a.R, idx, rv);
                    }
#pragma unroll
                    for (int q = 0; q < V; ++q) {
                        if (up[q]) xv[q] = fma(alpha[q], pv[q], xv[q]);
                        if (on[q]) pv[q] = fma(beta[q], pv[q], rv[q]);
                    }
                    if constexpr (decltype(kept_x)::value) stv<V>(K.x, at, xv);
                    else stv<V>(a.X, idx, xv);
                    if (any_on) stv<V>(a.P, idx, pv);
                });
        }
        if (!S.any) break;       // the x updates above reach the team at the next barrier
        if (!team_sync<NT>(a, first, T, ++episode, S)) return false;
    }

    // the x kept in LDS; b = 0: the solution is x = 0
    if (kept && lane_on)
        for (int64_t row = lo + rsub; row < lo + K.nx; row += RS) {
            double xv[V];
            ldv<V>(K.x, (row - lo) * nr + j0, xv);
            stv<V>(a.X, row * nr + j0, xv);
        }
    if (lane_on)
        for (int64_t row = lo + rsub; row < hi; row += RS)
#pragma unroll
            for (int q = 0; q < V; ++q)
                if (S.zero_b[j0 + q]) a.X[row * nr + j0 + q] = 0.0;
    if (!team_sync<NT>(a, first, T, ++episode, S)) return false;
    // true residual ||b - A x||^2
    {
        double acc[V];
#pragma unroll
        for (int q = 0; q < V; ++q) acc[q] = 0.0;
        if (lane_on)
            for (int64_t row = lo + rsub; row < hi; row += RS) {
                const int64_t idx = row * nr + j0;
                double s[V], bv[V];
                row_dot<V>(a, row, a.X, nr, j0, s);
                ldv<V>(a.B, idx, bv);
#pragma unroll
                for (int q = 0; q < V; ++q) {
                    const double rv = bv[q] - s[q];
                    acc[q] = fma(rv, rv, acc[q]);
                }
            }
        const double tr = wg_partial<NT, V>(acc, lanes, S);
        if (!team_sum<NT>(a, first, T, kSlotTrue, ++episode, tr, S)) return false;
    }
    if (rank == 0) {
        if (threadIdx.x < nr) {
            const int t = threadIdx.x;
            const double bn = sqrt(S.bb[t]);
            BatchOutDev o;
            o.status = S.status[t];
            o.iterations = S.iter[t];
            o.rel_res_recur = S.zero_b[t] ? 0.0 : sqrt(S.rr_last[t]) / bn;
            o.rel_res_true = S.zero_b[t] ? 0.0 : sqrt(S.sum[t]) / bn;
            a.out[(int64_t)sys * nr + t] = o;
        }
        if (threadIdx.x == 0) a.episodes[sys] = episode;
    }
    return true;
}

// Each workgroup solves its list of systems one after another: a member of a
// team of several workgroups has one, a workgroup hosting small systems
// (teams of one) several, so their rows share workgroups instead of each
// taking one.
template <int NT, int U, int V, int E>
__global__ __launch_bounds__(NT) void k_batch_cg(BatchArgs a) {
    __shared__ Shared<NT> S;
    if (threadIdx.x == 0) S.ok = 1;
    const int i0 = __builtin_amdgcn_readfirstlane(a.wg_item[blockIdx.x]);
    const int i1 = __builtin_amdgcn_readfirstlane(a.wg_item[blockIdx.x + 1]);
    for (int it = i0; it < i1; ++it) {
        const int sys = __builtin_amdgcn_readfirstlane(a.item_sys[it]);
        const int rank = __builtin_amdgcn_readfirstlane(a.item_rank[it]);
        if (!batch_solve_one<NT, U, V, E>(a, sys, rank, S)) return;
        __syncthreads();   // S is set up afresh by the next system
    }
}

const void *kernel_of(const BatchVariant &k) {
#define CGMI_BATCH(NT, U, V)                                                                   \
    if (k.threads == NT && k.rows_per_thread == U && k.rhs_per_lane == V)                      \
    return k.row_max <= 5 ? reinterpret_cast<const void *>(k_batch_cg<NT, U, V, 5>)            \
                          : reinterpret_cast<const void *>(k_batch_cg<NT, U, V, 6>)
    CGMI_BATCH(256, 1, 1);
    CGMI_BATCH(256, 1, 2);
    CGMI_BATCH(256, 2, 1);
    CGMI_BATCH(256, 2, 2);
    CGMI_BATCH(1024, 1, 1);
    CGMI_BATCH(1024, 1, 2);
    CGMI_BATCH(1024, 2, 1);
    CGMI_BATCH(1024, 2, 2);
#undef CGMI_BATCH
    return nullptr;
}

}  // namespace

int batch_blocks_per_cu(const BatchVariant &k) {
    int nb = 0;
    const void *fn = kernel_of(k);
    const int threads = k.threads, lds = batch_keep(threads) * (int)sizeof(double);
    if (!fn || (lds && hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess)) return 0;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fn, threads, lds) == hipSuccess ? nb : 0;
}

hipError_t launch_batch_cg(const BatchArgs &a, int grid, const BatchVariant &k, int cooperative, hipStream_t s) {
    if (grid <= 0) return hipSuccess;
    BatchArgs args = a;
    void *params[] = {&args};
    const void *fn = kernel_of(k);
    const int threads = k.threads;
    if (!fn) return hipErrorInvalidValue;
    args.keep = batch_keep(threads);
    args.lane_bits = 0;
    while ((k.rhs_per_lane << args.lane_bits) < a.nrhs) ++args.lane_bits;
    const unsigned lds = (unsigned)(args.keep * sizeof(double));
    if (lds) {
        const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    if (cooperative) return hipLaunchCooperativeKernel(fn, dim3(grid), dim3(threads), params, lds, s);
    // ordinary launch of a grid the caller has checked to be resident (the
    // team waits give up after their time limit if it were not)
    return hipLaunchKernel(fn, dim3(grid), dim3(threads), params, lds, s);
}

}  // namespace cgmi
