// kernels_resident.hip -- the whole of Algorithm 1 in one cooperative launch
// for systems above one workgroup's size whose rows fit the GPU's threads, one
// each (gfx950).
//
// With two kernels per iteration such a system spends most of an iteration
// between kernels: launches, and a first and last wave of loads that nothing
// overlaps (us per iteration, two kernels and here: 4200 rows of 5 entries 9.7
// and 4.5, 20K 9.3 and 4.6, 62K 9.4 and 4.8, 262K 12.5 and 6.5; of 7 entries,
// 32K rows 9.6 and 5.3, 262K 12.7 and 7.0).  What remains is two trips of the
// sums through memory, 1.5 to 2.5 us each, and one of r.  Here thread t of workgroup w owns row w NT + t for the whole
// solve and keeps its entries, x, r, p and q in registers, p also in LDS for
// its workgroup.  What crosses workgroups is the residual, written through to
// memory by its owner, and the partial sums.  A thread keeps its own copy of p
// for every column of another workgroup and advances it as the owner does,
// p = r + beta p, from the r it reads there, so p itself is never exchanged
// and an iteration has two waits: for the sum p^T q, and for r^T r, behind
// which every r is visible.
//
// Partial sums travel in 64-bit words that carry half of a value beside the
// number of the sum, so a reader knows a word as the one it waits for without
// any ordering between words, and no cache is written back or invalidated:
// r is stored and loaded with agent-scope atomics, which act beyond the XCDs'
// L2 caches, and every wave waits for its stores before its workgroup's sum
// is posted.  (r in such words too, needing no wait and loaded while r^T r is
// still being summed, gained nothing at 20K rows and lost 1.4 us per iteration
// at 262K, for twice the bytes.)  Waits are bounded by a wall-clock limit; on
// expiry the error flag ends every workgroup, and the host makes the solve with
// the separate kernels.
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>
#include <climits>
#include <cstdlib>
#include <type_traits>

#include "cg_device.h"
#include "cgmi_internal.h"

namespace cgmi {

namespace {

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

// Sum over each row of 16 lanes, the same value in all of them.
__device__ __forceinline__ double row_allsum(double v) {
    v += dpp_f64<0xB1>(v);   // quad_perm [1,0,3,2]
    v += dpp_f64<0x4E>(v);   // quad_perm [2,3,0,1]
    v += dpp_f64<0x141>(v);  // row_half_mirror
    v += dpp_f64<0x140>(v);  // row_mirror
    return v;
}

// Sum over the wave, the same value in every lane, in a fixed order.
__device__ __forceinline__ double wave_allsum(double v) {
    v = row_allsum(v);
    return (readlane_f64(v, 0) + readlane_f64(v, 16)) + (readlane_f64(v, 32) + readlane_f64(v, 48));
}

// Element i of an array of 8-byte values below 2^32 bytes: a 32-bit offset
// from the uniform base, where an index would cost a 64-bit address per lane.
template <class T>
__device__ __forceinline__ T *elem(T *base, uint32_t i) {
    typedef typename std::conditional<std::is_const<T>::value, const char, char>::type Byte;
    return reinterpret_cast<T *>(reinterpret_cast<Byte *>(base) + (uint32_t)(i * 8u));
}
__device__ __forceinline__ double load_agent(const double *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_agent(double *p, double v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

constexpr int kNT = 1024;   // threads of a workgroup: one workgroup per compute unit

template <int NT>
struct ResidentShared {
    double red[2][NT / kWave];
    double sum[2];
    int ok;
};

// One word of a pair: half of the bits of a value beside a tag.
__device__ __forceinline__ void store_pair(uint64_t *lo, uint64_t *hi, double v, uint32_t tag) {
    const uint64_t bits = (uint64_t)__double_as_longlong(v), t = (uint64_t)tag << 32;
    __hip_atomic_store(lo, t | (bits & 0xFFFFFFFFu), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(hi, t | bits >> 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t load_word(const uint64_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool tagged(uint64_t lo, uint64_t hi, uint32_t tag) {
    return (uint32_t)(lo >> 32) == tag && (uint32_t)(hi >> 32) == tag;
}
__device__ __forceinline__ double pair_value(uint64_t lo, uint64_t hi) {
    return __longlong_as_double((long long)(hi << 32 | (lo & 0xFFFFFFFFu)));
}

// Spin `spin` of a wait that began at t0: false when the launch is being
// abandoned (looked at every 64 spins).
__device__ __forceinline__ bool wait_on(const ResidentArgs &a, int spin, uint64_t t0, int64_t limit) {
    if ((spin & 63) != 63) return true;
    if (__hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return false;
    if ((int64_t)(wall_clock64() - t0) <= limit) return true;
    __hip_atomic_store(a.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return false;
}

// Sum of v over the grid, the same bits in every thread, in a fixed order.
// `no` counts the launch's sums from 1; consecutive sums alternate between two
// sets of words, so a set is written again only after its writer has seen
// every workgroup's word of the sum between, hence after every workgroup has
// read it.  Each workgroup posts its word in kResidentCopies copies and reads
// one of them, so that a copy's lines have 1/8 of the grid for readers (one
// copy: 9.5 us per iteration of 64^3 rows, 8: 7.7, 16: 8.2).  STORED: what any
// thread stored with store_agent before is visible to load_agent behind the
// sum.  False when the launch is being abandoned.
template <int NT, bool STORED>
__device__ __forceinline__ bool grid_sum(const ResidentArgs &a, double v, uint32_t no, ResidentShared<NT> &S,
                                         double &out) {
    constexpr int C = kResidentCopies, W = NT / kWave;
    static_assert(W <= 16 && C <= kWave, "one row of lanes sums the waves");
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave, half = no & 1;
    const int T = gridDim.x;
    if (STORED) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's stores are done
    v = wave_allsum(v);
    if (lane == 0) S.red[half][w] = v;
    __syncthreads();
    if (w == 0) {
        double s = row_allsum((lane & 15) < W ? S.red[half][lane & 15] : 0.0);
        if (lane < C) {
            uint64_t *const lo = a.words + ((size_t)half * C + lane) * 2 * T;
            store_pair(lo + blockIdx.x, lo + T + blockIdx.x, s, no);
        }
        const uint64_t *const lo = a.words + ((size_t)half * C + blockIdx.x % C) * 2 * T, *const hi = lo + T;
        constexpr int Q = kResidentMaxGroups / kWave;   // members per lane
        uint64_t l[Q], h[Q];
        int first = lane;
        asm volatile("" : "+v"(first));   // its addresses: worked out here, not kept
        bool ok = true;
        const uint64_t t0 = wall_clock64();
        for (int spin = 0;; ++spin) {
            bool all = true;
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if (q * kWave < T) {
                    const int m = min(first + q * kWave, T - 1);
                    l[q] = load_word(elem(lo, m));
                    h[q] = load_word(elem(hi, m));
                }
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if (q * kWave < T) all &= tagged(l[q], h[q], no);
            if (__all(all)) break;
            if (!__all(wait_on(a, spin, t0, no == 1 ? a.start_ticks : a.timeout_ticks))) {
                ok = false;
                break;
            }
        }
        s = 0.0;
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (lane + q * kWave < T) s += pair_value(l[q], h[q]);
        s = wave_allsum(s);
        if (lane == 0) {
            S.sum[half] = s;
            if (!ok) S.ok = 0;
        }
    }
    __syncthreads();
    out = S.sum[half];
    return S.ok != 0;
}

// W: entries of a row at most.
template <int NT, int W>
__global__ __launch_bounds__(NT) void k_cg_resident(ResidentArgs a) {
    __shared__ double s_p[NT];
    __shared__ ResidentShared<NT> S;
    if (threadIdx.x == 0) S.ok = 1;
    if (blockIdx.x == 0 && threadIdx.x == 0) a.st->done = kDoneRunning;   // left so by an abandoned launch
    const int n = a.n, lo = blockIdx.x * NT, i = lo + threadIdx.x;
    const bool mine = i < n;
    // the row's entries in CSR order; past its end the row itself with value 0
    int col[W];
    double v[W];
    const int beg = mine ? a.rp[i] : 0, len = mine ? a.rp[i + 1] - beg : 0;
#pragma unroll
    for (int e = 0; e < W; ++e) {
        col[e] = e < len ? a.ci[beg + e] : min(i, n - 1);
        v[e] = e < len ? a.val[beg + e] : 0.0;
    }
    auto away = [&](int e) { return (uint32_t)(col[e] - lo) >= (uint32_t)NT; };   // another workgroup's
    double x = 0.0, r = 0.0, p = 0.0, bi = 0.0;
    if (mine) {
        double s = 0.0;
#pragma unroll
        for (int e = 0; e < W; ++e) s = fma(v[e], *elem(a.x, col[e]), s);
        x = a.x[i];
        bi = a.b[i];
        r = bi - s;
        store_agent(elem(a.r, i), r);
    }
    uint32_t no = 1;
    double rho, bb;
    if (!grid_sum<NT, true>(a, r * r, no++, S, rho)) return;
    if (!grid_sum<NT, false>(a, bi * bi, no++, S, bb)) return;
    if (bb == 0.0) {   // b = 0: the solution is x = 0
        if (mine) a.x[i] = 0.0;
        if (i == 0) {
            a.st->iter = 0;
            a.st->done = kDoneConverged;
            a.st->rho[0] = a.st->rr = a.st->bb = a.st->rr_true = 0.0;
        }
        return;
    }
    double pn[W];   // p of other workgroups' columns
#pragma unroll
    for (int e = 0; e < W; ++e) pn[e] = away(e) ? load_agent(elem(a.r, col[e])) : 0.0;
    p = r;
    int status = kDoneMaxit, k = 0;
    for (;;) {
        if (stop_test(rho, bb, a.tol)) {
            status = kDoneConverged;
            break;
        }
        if (k >= a.maxit) break;
        s_p[threadIdx.x] = p;
        __syncthreads();
        double q = 0.0;
#pragma unroll
        for (int e = 0; e < W; ++e) q = fma(v[e], away(e) ? pn[e] : s_p[(uint32_t)(col[e] - lo) % NT], q);
        double pq;
        if (!grid_sum<NT, false>(a, p * q, no++, S, pq)) return;
        if (!(pq > 0.0) || !isfinite(pq)) {
            status = kDoneBreakdown;
            break;
        }
        const double alpha = rho / pq;
        x = fma(alpha, p, x);
        r = fma(-alpha, q, r);
        ++k;
        if (mine) store_agent(elem(a.r, i), r);
        double rr;
        if (!grid_sum<NT, true>(a, r * r, no++, S, rr)) return;
        const double beta = rr / rho;
        rho = rr;
        p = fma(beta, p, r);
        // (columns made opaque: their addresses and masks, worked out once
        // before the loop and kept, would not fit the registers)
#pragma unroll
        for (int e = 0; e < W; ++e) asm volatile("" : "+v"(col[e]));
#pragma unroll
        for (int e = 0; e < W; ++e)
            if (away(e)) pn[e] = fma(beta, pn[e], load_agent(elem(a.r, col[e])));
    }
    // the solution, and the true residual b - A x
    if (mine) store_agent(elem(a.x, i), x);
    double rr_true;
    if (!grid_sum<NT, true>(a, 0.0, no++, S, rr_true)) return;
    double s = 0.0;
    if (mine) {
#pragma unroll
        for (int e = 0; e < W; ++e) s = fma(v[e], load_agent(elem(a.x, col[e])), s);
        s = a.b[i] - s;
    }
    if (!grid_sum<NT, false>(a, s * s, no++, S, rr_true)) return;
    if (i == 0) {
        a.st->iter = k;
        a.st->done = status;
        a.st->rho[0] = a.st->rr = rho;
        a.st->bb = bb;
        a.st->rr_true = rr_true;
    }
}

// The same for a global stencil (StenGlobal), several rows per thread: a
// workgroup's M consecutive rows keep x, r and q in registers, row u NT + ...
// of a thread in slice order, and in LDS p of every column they have: the rows
// moved by each offset, overlapping ranges in one segment.  What lies outside
// the workgroup's rows there are its copies of other workgroups' p.  Constant values are launch arguments, so
// an iteration then touches memory for r alone, and of r only the rows that
// others read; other values are streamed from the stencil slices.  Us per
// iteration, separate kernels (whose vectors pass through memory in every one)
// and here: 2-D diffusion 1024^2 26.6 and 12.3, 1500 x 1401 43.0 and 21.7 (84
// MB of values, 13 us at 6.4 TB/s), 1600^2 51 and 24; Poisson 1024^2 21.4 and
// 9.7, 1500 x 1400 33.7 and 15.9, 72^3 16.3 and 10.0, 90^3 19.4 and 14.2.
template <int NT, int RPT, int W, bool KONST>
__global__ __launch_bounds__(NT) void k_cg_window(ResidentArgs a, WindowArgs g) {
    extern __shared__ double s_p[];   // [g.entries]
    __shared__ ResidentShared<NT> S;
    if (threadIdx.x == 0) S.ok = 1;
    if (blockIdx.x == 0 && threadIdx.x == 0) a.st->done = kDoneRunning;   // left so by an abandoned launch
    const int n = a.n, lo = blockIdx.x * g.rows, end = min(n, lo + g.rows);
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    // the thread's row u; its first one is made opaque before every phase, or
    // the addresses of all rows would be worked out once and kept in registers
    int row0 = lo + w * kWave + lane;
    auto row_of = [&](int u) { return row0 + u * NT; };
    // whether another workgroup's rows have this one as a column
    auto shared = [&](int i) { return i - lo < g.head || i - lo >= g.tail; };
    auto phase = [&] { asm volatile("" : "+v"(row0)); };
    // a row's entries (constant ones: which it has); loaded for every row, so
    // that the loads in flight can be counted, but past the end all lanes read
    // one place (the rows there are the next workgroup's)
    struct Entries {
        double v[KONST ? 1 : W];
        uint32_t have;
    };
    auto entries = [&](int i) {
        Entries E;
        if (KONST) {
            E.have = g.mask[i < end ? i : 0];
        } else {
            const double *const v = g.val + (i < end ? (int64_t)(i / kWave) * (W * kWave) + lane : 0);
#pragma unroll
            for (int e = 0; e < W; ++e) E.v[KONST ? 0 : e] = v[e * kWave];
        }
        return E;
    };
    // q of a row from the window, its products and sums rounded in turn
    auto product = [&](int i, const Entries &E) {
        const double *const at = s_p + (i - lo);
        double s = 0.0;
#pragma unroll
        for (int e = 0; e < W; ++e)
            s = add_rounded(s, KONST ? ((E.have >> e) & 1u ? g.sten.val[e] : 0.0) : E.v[KONST ? 0 : e], at[g.disp[e]]);
        return s;
    };
    // f(u, row, q) of the thread's rows, the next row's entries on their way;
    // first: those of row 0
    auto for_products = [&](const Entries &first, auto f) {
        Entries E = first;
#pragma unroll
        for (int u = 0; u < RPT; ++u) {
            const Entries cur = E;
            if (u + 1 < RPT) E = entries(row_of(u + 1));
            if (row_of(u) < end) f(u, row_of(u), product(row_of(u), cur));
        }
    };
    // sets the window's entries outside the workgroup's rows to f(old entry, v
    // of its column), four loads of v in flight per thread
    auto update_ends = [&](const double *v, auto f) {
        for (int sg = 0; sg < g.nseg; ++sg) {
            const int first = lo + g.seg[sg].start, len = g.seg[sg].len;
            double *const at = s_p + g.seg[sg].base;
            auto other = [&](int k, int c) {
                return k < len && c >= 0 && c < n && (uint32_t)(c - lo) >= (uint32_t)g.rows;
            };
            for (int k0 = threadIdx.x; k0 < len; k0 += 4 * NT) {
                double x4[4];
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (other(k0 + j * NT, first + k0 + j * NT)) x4[j] = load_agent(elem(v, first + k0 + j * NT));
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (other(k0 + j * NT, first + k0 + j * NT)) at[k0 + j * NT] = f(at[k0 + j * NT], x4[j]);
            }
        }
    };
    for (int sg = 0; sg < g.nseg; ++sg)
        for (int k = threadIdx.x; k < g.seg[sg].len; k += NT) {
            const int c = lo + g.seg[sg].start + k;
            s_p[g.seg[sg].base + k] = c >= 0 && c < n ? a.x[c] : 0.0;
        }
    __syncthreads();
    double x[RPT], r[RPT], q[RPT];
    double acc = 0.0, accb = 0.0;
#pragma unroll
    for (int u = 0; u < RPT; ++u) x[u] = r[u] = q[u] = 0.0;
    for_products(entries(row_of(0)), [&](int u, int i, double s) {
        const double bi = a.b[i];
        x[u] = s_p[i - lo + g.own];
        r[u] = bi - s;
        acc = fma(r[u], r[u], acc);
        accb = fma(bi, bi, accb);
        if (shared(i)) store_agent(elem(a.r, i), r[u]);
    });
    uint32_t no = 1;
    double rho, bb;
    if (!grid_sum<NT, true>(a, acc, no++, S, rho)) return;
    if (!grid_sum<NT, false>(a, accb, no++, S, bb)) return;
    if (bb == 0.0) {   // b = 0: the solution is x = 0
#pragma unroll
        for (int u = 0; u < RPT; ++u)
            if (row_of(u) < end) a.x[row_of(u)] = 0.0;
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            a.st->iter = 0;
            a.st->done = kDoneConverged;
            a.st->rho[0] = a.st->rr = a.st->bb = a.st->rr_true = 0.0;
        }
        return;
    }
    // p = r: every read of x in the window is behind a barrier
    phase();
#pragma unroll
    for (int u = 0; u < RPT; ++u)
        if (row_of(u) < end) s_p[row_of(u) - lo + g.own] = r[u];
    update_ends(a.r, [](double, double v) { return v; });
    int status = kDoneMaxit, k = 0;
    Entries first = entries(row_of(0));
    for (;;) {
        if (stop_test(rho, bb, a.tol)) {
            status = kDoneConverged;
            break;
        }
        if (k >= a.maxit) break;
        __syncthreads();
        acc = 0.0;
        phase();
        for_products(first, [&](int u, int i, double s) {
            q[u] = s;
            acc = fma(s_p[i - lo + g.own], s, acc);
        });
        double pq;
        if (!grid_sum<NT, false>(a, acc, no++, S, pq)) return;
        if (!(pq > 0.0) || !isfinite(pq)) {
            status = kDoneBreakdown;
            break;
        }
        const double alpha = rho / pq;
        acc = 0.0;
        phase();
#pragma unroll
        for (int u = 0; u < RPT; ++u) {
            const int i = row_of(u);
            if (i < end) {
                x[u] = fma(alpha, s_p[i - lo + g.own], x[u]);
                r[u] = fma(-alpha, q[u], r[u]);
                acc = fma(r[u], r[u], acc);
                if (shared(i)) store_agent(elem(a.r, i), r[u]);
            }
        }
        ++k;
        first = entries(row_of(0));   // under way during the sum
        double rr;
        if (!grid_sum<NT, true>(a, acc, no++, S, rr)) return;
        const double beta = rr / rho;
        rho = rr;
        update_ends(a.r, [beta](double p, double v) { return fma(beta, p, v); });
        phase();
#pragma unroll
        for (int u = 0; u < RPT; ++u) {
            const int i = row_of(u);
            if (i < end) {
                double &p = s_p[i - lo + g.own];
                p = fma(beta, p, r[u]);
            }
        }
    }
    // the solution, and the true residual b - A x
    phase();
#pragma unroll
    for (int u = 0; u < RPT; ++u)
        if (row_of(u) < end) store_agent(elem(a.x, row_of(u)), x[u]);
    double rr_true;
    if (!grid_sum<NT, true>(a, 0.0, no++, S, rr_true)) return;
    phase();
#pragma unroll
    for (int u = 0; u < RPT; ++u)
        if (row_of(u) < end) s_p[row_of(u) - lo + g.own] = x[u];
    update_ends(a.x, [](double, double v) { return v; });
    __syncthreads();
    acc = 0.0;
    phase();
    for_products(entries(row_of(0)), [&](int, int i, double s) {
        const double v = a.b[i] - s;
        acc = fma(v, v, acc);
    });
    if (!grid_sum<NT, false>(a, acc, no++, S, rr_true)) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.st->iter = k;
        a.st->done = status;
        a.st->rho[0] = a.st->rr = rho;
        a.st->bb = bb;
        a.st->rr_true = rr_true;
    }
}

// Preconditioned CG, z = G^T (G r), for a 5-point A with a factor on its lower
// part, as above with three sums per iteration: p^T q, r^T r (behind it the r
// of other workgroups) and r^T z (their z, from which the copies of p outside
// the workgroup's rows advance).  One window holds p, another r and, once it
// has been used, t = G r; t of the rows above the workgroup's, which G^T needs,
// is computed again here.  Us per iteration, three kernels and here: 1024^2
// diffusion 43.5 and 23.7 (98 MB of values, 15 us at 6.4 TB/s), 777 x 700 31.9
// and 18.4, 1300^2 73.6 and 32.4, 150 x 133 17.1 and 8.5.
template <int RPT, bool KONST>
__global__ __launch_bounds__(kNT) void k_pcg_window(ResidentArgs a, PcgWindowArgs g) {
    constexpr int W = 5, RT = RPT + kPcgReach / kNT;   // rows of t: the reach more
    extern __shared__ double lds[];   // two windows of g.rows + 2 g.reach
    __shared__ ResidentShared<kNT> S;
    if (threadIdx.x == 0) S.ok = 1;
    if (blockIdx.x == 0 && threadIdx.x == 0) a.st->done = kDoneRunning;   // left so by an abandoned launch
    const int n = a.n, lo = blockIdx.x * g.rows, end = min(n, lo + g.rows), t_end = min(n, lo + g.rows + g.reach);
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave, window = g.rows + 2 * g.reach;
    double *const s_p = lds, *const s_r = lds + window;
    int row0 = lo + w * kWave + lane;   // as in k_cg_window
    auto row_of = [&](int u) { return row0 + u * kNT; };
    auto phase = [&] { asm volatile("" : "+v"(row0)); };
    auto shared = [&](int i) { return i - lo < g.reach || i - lo >= g.rows - g.reach; };
    auto at = [&](double *win, int i) -> double & { return win[i - lo + g.reach]; };
    // sets the entries of a window outside the workgroup's rows to f(old, v)
    auto update_ends = [&](double *win, const double *v, auto f) {
        for (int k0 = threadIdx.x; k0 < 2 * g.reach; k0 += 4 * kNT) {
            double x4[4];
            auto col = [&](int j) {
                const int k = k0 + j * kNT;
                return k < g.reach ? lo - g.reach + k : lo + g.rows + k - g.reach;
            };
            auto other = [&](int j) { return k0 + j * kNT < 2 * g.reach && col(j) >= 0 && col(j) < n; };
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (other(j)) x4[j] = load_agent(elem(v, col(j)));
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (other(j)) at(win, col(j)) = f(at(win, col(j)), x4[j]);
        }
    };
    struct Slots {
        double v[W];
        uint32_t have;
    };
    auto slots = [&](const double *val, int width, int i, int limit) {   // as entries in k_cg_window (777 x 700: 23.2 to 18.4)
        Slots E;
        const double *const v = val + (i < limit ? (int64_t)(i / kWave) * (width * kWave) + lane : 0);
#pragma unroll
        for (int e = 0; e < W; ++e)
            if (e < width) E.v[e] = v[e * kWave];
        return E;
    };
    auto a_slots = [&](int i) {
        if (!KONST) return slots(g.val, W, i, end);
        Slots E;
        E.have = g.mask[i < end ? i : 0];
#pragma unroll
        for (int e = 0; e < W; ++e) E.v[e] = (E.have >> e) & 1u ? g.sten.val[e] : 0.0;
        return E;
    };
    auto g_slots = [&](int i) { return slots(g.g_val, 3, i, t_end); };
    auto gt_slots = [&](int i) { return slots(g.gt_val, 3, i, end); };
    auto dot = [&](const Slots &E, int width, const int32_t *offs, double *win, int i) {
        double s = 0.0;
#pragma unroll
        for (int e = 0; e < W; ++e)
            if (e < width) s = add_rounded(s, E.v[e], at(win, i + offs[e]));
        return s;
    };
    // z = G^T (G r) of the workgroup's rows into z, r^T z into acc; r of the
    // window's ends is read behind the sum before.  first: G's slots of row 0
    double x[RPT], r[RPT], z[RPT];
    double acc = 0.0;
    auto precondition = [&](const Slots &first) {
        update_ends(s_r, a.r, [](double, double v) { return v; });
        phase();
#pragma unroll
        for (int u = 0; u < RPT; ++u)
            if (row_of(u) < end) at(s_r, row_of(u)) = r[u];
        __syncthreads();
        double t[RT];
        Slots E = first;
        phase();
#pragma unroll
        for (int u = 0; u < RT; ++u) {
            const Slots cur = E;
            if (u + 1 < RT) E = g_slots(row_of(u + 1));
            t[u] = row_of(u) < t_end ? dot(cur, 3, g.g_offs, s_r, row_of(u)) : 0.0;
        }
        E = gt_slots(row_of(0));
        __syncthreads();
        phase();
#pragma unroll
        for (int u = 0; u < RT; ++u)
            if (row_of(u) < t_end) at(s_r, row_of(u)) = t[u];
        __syncthreads();
        acc = 0.0;
        phase();
#pragma unroll
        for (int u = 0; u < RPT; ++u) {
            const Slots cur = E;
            if (u + 1 < RPT) E = gt_slots(row_of(u + 1));
            const int i = row_of(u);
            if (i < end) {
                z[u] = dot(cur, 3, g.gt_offs, s_r, i);
                acc = fma(r[u], z[u], acc);
                if (shared(i)) store_agent(elem(g.z, i), z[u]);
            }
        }
    };
    for (int k = threadIdx.x; k < window; k += kNT) {
        const int c = lo - g.reach + k;
        s_p[k] = c >= 0 && c < n ? a.x[c] : 0.0;
        s_r[k] = 0.0;
    }
    __syncthreads();
    double accb = 0.0;
#pragma unroll
    for (int u = 0; u < RPT; ++u) {
        const int i = row_of(u);
        x[u] = r[u] = z[u] = 0.0;
        if (i < end) {
            const double bi = a.b[i];
            x[u] = at(s_p, i);
            r[u] = bi - dot(a_slots(i), W, g.sten.offs, s_p, i);
            acc = fma(r[u], r[u], acc);
            accb = fma(bi, bi, accb);
            if (shared(i)) store_agent(elem(a.r, i), r[u]);
        }
    }
    uint32_t no = 1;
    double rr, bb, rho;
    if (!grid_sum<kNT, true>(a, acc, no++, S, rr)) return;
    if (!grid_sum<kNT, false>(a, accb, no++, S, bb)) return;
    precondition(g_slots(row_of(0)));
    if (!grid_sum<kNT, true>(a, acc, no++, S, rho)) return;
    // p = z
    phase();
#pragma unroll
    for (int u = 0; u < RPT; ++u)
        if (row_of(u) < end) at(s_p, row_of(u)) = z[u];
    update_ends(s_p, g.z, [](double, double v) { return v; });
    int status = kDoneRunning, k = 0;
    if (stop_test(rr, bb, a.tol) || bb == 0.0) status = kDoneConverged;
    else if (a.maxit <= 0) status = kDoneMaxit;
    Slots first = a_slots(row_of(0));
    while (status == kDoneRunning) {
        __syncthreads();
        double q[RPT];
        acc = 0.0;
        phase();
#pragma unroll
        for (int u = 0; u < RPT; ++u) {
            const Slots cur = first;
            if (u + 1 < RPT) first = a_slots(row_of(u + 1));
            const int i = row_of(u);
            q[u] = 0.0;
            if (i < end) {
                q[u] = dot(cur, W, g.sten.offs, s_p, i);
                acc = fma(at(s_p, i), q[u], acc);
            }
        }
        double pq;
        if (!grid_sum<kNT, false>(a, acc, no++, S, pq)) return;
        if (!(pq > 0.0) || !isfinite(pq)) {
            status = kDoneBreakdown;
            break;
        }
        const double alpha = rho / pq;
        acc = 0.0;
        phase();
#pragma unroll
        for (int u = 0; u < RPT; ++u) {
            const int i = row_of(u);
            if (i < end) {
                x[u] = fma(alpha, at(s_p, i), x[u]);
                r[u] = fma(-alpha, q[u], r[u]);
                acc = fma(r[u], r[u], acc);
                if (shared(i)) store_agent(elem(a.r, i), r[u]);
            }
        }
        ++k;
        const Slots g0 = g_slots(row_of(0));   // under way during the sum
        if (!grid_sum<kNT, true>(a, acc, no++, S, rr)) return;
        precondition(g0);
        first = a_slots(row_of(0));
        double rz;
        if (!grid_sum<kNT, true>(a, acc, no++, S, rz)) return;
        const double beta = rz / rho;
        rho = rz;
        if ((!(rz > 0.0) || !isfinite(rz)) && rr != 0.0) status = kDoneBreakdown;
        else if (stop_test(rr, bb, a.tol)) status = kDoneConverged;
        else if (k >= a.maxit) status = kDoneMaxit;
        if (status != kDoneRunning) break;
        update_ends(s_p, g.z, [beta](double p, double v) { return fma(beta, p, v); });
        phase();
#pragma unroll
        for (int u = 0; u < RPT; ++u)
            if (row_of(u) < end) at(s_p, row_of(u)) = fma(beta, at(s_p, row_of(u)), z[u]);
    }
    // b = 0: the solution is x = 0; after a breakdown x stays as it was given
    double rr_true = 0.0;
    if (status != kDoneBreakdown) {
        phase();
#pragma unroll
        for (int u = 0; u < RPT; ++u)
            if (row_of(u) < end) store_agent(elem(a.x, row_of(u)), bb == 0.0 ? 0.0 : x[u]);
        if (!grid_sum<kNT, true>(a, 0.0, no++, S, rr_true)) return;
        phase();
#pragma unroll
        for (int u = 0; u < RPT; ++u)
            if (row_of(u) < end) at(s_p, row_of(u)) = x[u];
        update_ends(s_p, a.x, [](double, double v) { return v; });
        __syncthreads();
        acc = 0.0;
        phase();
#pragma unroll
        for (int u = 0; u < RPT; ++u) {
            const int i = row_of(u);
            if (i < end) {
                const double v = a.b[i] - dot(a_slots(i), W, g.sten.offs, s_p, i);
                acc = fma(v, v, acc);
            }
        }
        if (!grid_sum<kNT, false>(a, acc, no++, S, rr_true)) return;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.st->iter = k;
        a.st->done = status;
        a.st->rho[0] = rho;
        a.st->rr = rr;
        a.st->bb = bb;
        a.st->rr_true = rr_true;
    }
}

const void *pcg_window_fn(int rows, bool konst) {
#define CGMI_PCG_WINDOW(RPT)                                                            \
    if (rows <= kNT * RPT)                                                              \
    return konst ? reinterpret_cast<const void *>(k_pcg_window<RPT, true>)              \
                 : reinterpret_cast<const void *>(k_pcg_window<RPT, false>)
    CGMI_PCG_WINDOW(1);
    CGMI_PCG_WINDOW(2);
    CGMI_PCG_WINDOW(4);
    CGMI_PCG_WINDOW(6);
    CGMI_PCG_WINDOW(7);
#undef CGMI_PCG_WINDOW
    return nullptr;
}

struct WindowFn {
    const void *fn;
    int threads;
};

template <int W, bool KONST>
WindowFn window_fn_of(int rows) {
#define CGMI_WINDOW(NT, RPT) \
    if (rows <= NT * RPT) return {reinterpret_cast<const void *>(k_cg_window<NT, RPT, W, KONST>), NT}
    // 1024 threads as long as the rows fit their 128 registers; 512 lost to
    // them there (1024^2 diffusion 13.2 against 12.3 us per iteration) and won
    // beyond (1500 x 1401: 21.7 against 25.3 with 12 rows per thread, spilled)
    CGMI_WINDOW(1024, 2);
    CGMI_WINDOW(1024, 4);
    CGMI_WINDOW(1024, 6);
    CGMI_WINDOW(1024, 8);
    if constexpr (W <= 5) CGMI_WINDOW(512, 20);   // 7: its window does not fit LDS there
#undef CGMI_WINDOW
    return {nullptr, 0};
}

WindowFn window_fn(const StenGlobal &C, int rows) {
    if (C.width == 3) return C.konst ? window_fn_of<3, true>(rows) : window_fn_of<3, false>(rows);
    if (C.width == 5) return C.konst ? window_fn_of<5, true>(rows) : window_fn_of<5, false>(rows);
    if (C.width == 7) return C.konst ? window_fn_of<7, true>(rows) : window_fn_of<7, false>(rows);
    return {nullptr, 0};
}

const void *resident_fn(int max_row_len) {
    return max_row_len <= 5 ? reinterpret_cast<const void *>(k_cg_resident<kNT, 5>)
                            : reinterpret_cast<const void *>(k_cg_resident<kNT, kResidentMaxRow>);
}

}  // namespace

int resident_groups(int32_t n, int32_t max_row_len, int cus) {
    if (n <= 0 || max_row_len < 0 || max_row_len > kResidentMaxRow) return 0;
    const int groups = (n + kNT - 1) / kNT;
    return groups <= std::min(cus, kResidentMaxGroups) ? groups : 0;
}

hipError_t launch_cg_resident(const ResidentArgs &a, int32_t max_row_len, int cus, hipStream_t s) {
    const int groups = resident_groups(a.n, max_row_len, cus);
    if (!groups) return hipErrorInvalidValue;
    ResidentArgs args = a;
    void *params[] = {&args};
    return hipLaunchCooperativeKernel(resident_fn(max_row_len), dim3(groups), dim3(kNT), params, 0, s);
}

bool window_shape(int32_t n, const StenGlobal &C, int cus, WindowArgs &g) {
    if (n <= 0 || C.width == 0) return false;
    const int groups_max = std::min(cus, kResidentMaxGroups);
    const int64_t rows = std::max<int64_t>(1024, ((int64_t)(n + groups_max - 1) / groups_max + kWave - 1) / kWave * kWave);
    if (rows > kWindowEntries) return false;
    g.rows = (int32_t)rows;
    g.groups = (int32_t)((n + rows - 1) / rows);
    g.sten = C;
    if (!window_fn(C, g.rows).fn) return false;
    g.head = std::max(0, C.offs[C.width - 1]);
    g.tail = g.rows + std::min(0, C.offs[0]);
    // the rows moved by every offset, and the rows themselves; ascending
    int32_t moved[kSliceMaxWidth + 1];
    int count = 0;
    bool own = false;
    for (int e = 0; e < C.width; ++e) {
        if (!own && C.offs[e] >= 0) {
            if (C.offs[e] > 0) moved[count++] = 0;
            own = true;
        }
        moved[count++] = C.offs[e];
    }
    if (!own) moved[count++] = 0;
    g.nseg = 0;
    int64_t entries = 0;
    for (int k = 0; k < count; ++k) {
        WindowSegment *const last = g.nseg ? &g.seg[g.nseg - 1] : nullptr;
        if (last && moved[k] <= (int64_t)last->start + last->len) {
            entries += moved[k] + rows - ((int64_t)last->start + last->len);
            last->len = (int32_t)(moved[k] + rows - last->start);
        } else {
            if (entries > kWindowEntries) return false;
            g.seg[g.nseg++] = {moved[k], (int32_t)rows, (int32_t)entries};
            entries += rows;
        }
        const WindowSegment &in = g.seg[g.nseg - 1];
        const int32_t at = in.base + (moved[k] - in.start);
        if (moved[k] == 0) g.own = at;
        for (int e = 0; e < C.width; ++e)
            if (C.offs[e] == moved[k]) g.disp[e] = at;
    }
    g.entries = (int32_t)std::min<int64_t>(entries, INT32_MAX);
    return entries <= kWindowEntries;
}

hipError_t launch_cg_window(const ResidentArgs &a, const WindowArgs &g, hipStream_t s) {
    const WindowFn k = window_fn(g.sten, g.rows);
    if (!k.fn) return hipErrorInvalidValue;
    const size_t lds = sizeof(double) * (size_t)g.entries;
    const hipError_t e = hipFuncSetAttribute(k.fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    ResidentArgs args = a;
    WindowArgs gs = g;
    void *params[] = {&args, &gs};
    return hipLaunchCooperativeKernel(k.fn, dim3(g.groups), dim3(k.threads), params, (unsigned)lds, s);
}

bool pcg_window_shape(int32_t n, const StenGlobal &A, const StenGlobal &G, const StenGlobal &GT, int cus,
                      PcgWindowArgs &g) {
    if (n <= 0 || A.width != 5 || G.width != 3 || GT.width != 3 || G.konst || GT.konst) return false;
    int32_t reach = 0;
    for (int e = 0; e < 5; ++e) reach = std::max(reach, std::abs(A.offs[e]));
    for (int e = 0; e < 3; ++e) {
        if (G.offs[e] > 0 || GT.offs[e] != -G.offs[2 - e]) return false;
        reach = std::max(reach, -G.offs[e]);
    }
    if (reach > kPcgReach) return false;
    const int groups_max = std::min(cus, kResidentMaxGroups);
    const int64_t rows = std::max<int64_t>(kNT, ((int64_t)(n + groups_max - 1) / groups_max + kWave - 1) / kWave * kWave);
    if (2 * (rows + 2 * reach) > kWindowEntries || !pcg_window_fn((int)rows, A.konst != 0)) return false;
    g.sten = A;
    std::copy(G.offs, G.offs + 3, g.g_offs);
    std::copy(GT.offs, GT.offs + 3, g.gt_offs);
    g.rows = (int32_t)rows;
    g.reach = reach;
    g.groups = (int32_t)((n + rows - 1) / rows);
    return true;
}

hipError_t launch_pcg_window(const ResidentArgs &a, const PcgWindowArgs &g, hipStream_t s) {
    const void *fn = pcg_window_fn(g.rows, g.sten.konst != 0);
    if (!fn) return hipErrorInvalidValue;
    const size_t lds = 2 * sizeof(double) * ((size_t)g.rows + 2 * (size_t)g.reach);
    const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    ResidentArgs args = a;
    PcgWindowArgs gs = g;
    void *params[] = {&args, &gs};
    return hipLaunchCooperativeKernel(fn, dim3(g.groups), dim3(kNT), params, (unsigned)lds, s);
}

}  // namespace cgmi
