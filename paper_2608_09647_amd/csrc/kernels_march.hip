// kernels_march.hip -- products with a constant-coefficient 7-point operator
// on a grid larger than the caches, walked along its largest offset (gfx950).
//
// With the entries as launch arguments a product reads p and writes q, but
// every row gathers seven entries of p, and an L2 hit takes as much of a
// compute unit's memory path as a miss: 256^3 rows took 112 us, six passes
// over p in lines moved, against 50 for the bytes themselves.  Here a
// workgroup takes a tile of 2048 consecutive rows of one plane and walks it
// from plane to plane: the planes below and above a row are in the registers
// of its thread, its neighbours within the plane in LDS, where each plane of
// the tile is put once with the line before and after it.  So p is loaded
// once, and 25% more for the lines (of 256 rows) and 1/8 more for the planes
// at the ends of a walk of 16: 53 us, 5.0 TB/s for p and q.
//
// Rows are summed as by the other kernels: ascending columns, products and
// sums rounded in turn, absent entries left out.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "cg_device.h"

namespace cgmi {

namespace {

constexpr int kMT = 512;                   // threads
constexpr int kMPairs = 2;                 // pairs of rows per thread
constexpr int kMTile = kMT * kMPairs * 2;  // rows of a tile
constexpr int kMHalo = 2 * kMarchLine / kMT;   // entries before and behind the tile per thread

struct MarchShape {
    int32_t planes, tiles;     // of the grid; tiles of a plane
    int32_t walk, chunks;      // planes of a walk, walks of a tile
};

typedef double dbl2m __attribute__((ext_vector_type(2)));

// One row: its seven entries of p in column order, the ones it has in `have`.
// ENDS: only the two nearest in the line may be missing.
template <bool ENDS>
__device__ __forceinline__ double march_row(const StenGlobal &C, const double (&x)[7], uint32_t have) {
    double s = 0.0;
#pragma unroll
    for (int e = 0; e < 7; ++e) {
        const double t = add_rounded(s, C.val[e], x[e]);
        s = (ENDS && e != 2 && e != 4) || ((have >> e) & 1u) ? t : s;
    }
    return s;
}

template <int MODE>
__global__ __launch_bounds__(kMT, 4) void k_spmv_march(int32_t m, StenGlobal C, MarchShape G,
                                                       const uint8_t *__restrict__ mask, const double *__restrict__ p,
                                                       double *__restrict__ q, double *__restrict__ out,
                                                       const DevState *__restrict__ st) {
    extern __shared__ double win[];   // two planes of the tile with `line` entries on both sides
    __shared__ double sh[kMT / kWave];
    if (st && st->done) return;
    const int line = C.offs[5], plane = C.offs[6], near = C.offs[4], width = kMTile + 2 * line;
    const int items = G.tiles * G.chunks;
    double acc = 0.0;
    // neighbouring tiles on the same XCD (workgroups go round the eight)
    const int per = (items + 7) / 8;
    for (int w = blockIdx.x; w < 8 * per; w += gridDim.x) {
        const int item = (w & 7) * per + (w >> 3);
        if (item >= items) continue;   // (uniform, as every branch around a barrier here)
        const int chunk = item / G.tiles, t0 = (item - chunk * G.tiles) * kMTile;
        const int z0 = chunk * G.walk, z1 = min(G.planes, z0 + G.walk);
        // entry `at` of plane z, clamped to the vector (what is then read is
        // not the row's: its entry there is missing)
        auto index = [&](int z, int at) { return (int)min(max((int64_t)z * plane + at, (int64_t)0), (int64_t)m - 1); };
        auto load_rows = [&](int z, dbl2m (&v)[kMPairs]) {
#pragma unroll
            for (int k = 0; k < kMPairs; ++k) {
                const int i = min(index(z, t0 + 2 * (k * kMT + (int)threadIdx.x)), m - 2);
                __builtin_memcpy(&v[k], p + i, 16);
            }
        };
        auto load_halo = [&](int z, double (&h)[kMHalo]) {
#pragma unroll
            for (int k = 0; k < kMHalo; ++k) {
                const int j = k * kMT + (int)threadIdx.x;   // the line before, then the line behind
                h[k] = p[j < 2 * line ? index(z, j < line ? t0 - line + j : t0 + kMTile + j - line) : 0];
            }
        };
        auto load_mask = [&](int z, uint32_t (&v)[kMPairs]) {
#pragma unroll
            for (int k = 0; k < kMPairs; ++k) {
                const int i = min(index(z, t0 + 2 * (k * kMT + (int)threadIdx.x)), m - 2);
                uint16_t u;
                __builtin_memcpy(&u, mask + i, 2);
                v[k] = u;
            }
        };
        dbl2m below[kMPairs], own[kMPairs], above[kMPairs], next[kMPairs];
        double halo[kMHalo], halo_next[kMHalo];
        uint32_t have[kMPairs], have_next[kMPairs];
        load_rows(z0 - 1, below);
        load_rows(z0, own);
        load_halo(z0, halo);
        load_mask(z0, have);
        load_rows(z0 + 1, above);
        for (int z = z0; z < z1; ++z) {
            load_rows(z + 2, next);
            load_halo(z + 1, halo_next);
            load_mask(z + 1, have_next);
            double *const buf = win + (z & 1) * width;
#pragma unroll
            for (int k = 0; k < kMPairs; ++k) {
                double *const at = buf + line + 2 * (k * kMT + (int)threadIdx.x);
                at[0] = own[k].x;
                at[1] = own[k].y;
            }
#pragma unroll
            for (int k = 0; k < kMHalo; ++k) {
                const int j = k * kMT + (int)threadIdx.x;
                if (j < 2 * line) buf[j < line ? j : j + kMTile] = halo[k];
            }
            __syncthreads();   // and plane z - 2, read from this half, is done with
#pragma unroll
            for (int k = 0; k < kMPairs; ++k) {
                const int at = 2 * (k * kMT + (int)threadIdx.x);
                const int64_t i = (int64_t)z * plane + t0 + at;
                const bool in0 = t0 + at < plane && i < m, in1 = t0 + at + 1 < plane && i + 1 < m;
                const double *const b = buf + line + at;
                const double x0[7] = {below[k].x, b[-line], b[-near], own[k].x, b[near], b[line], above[k].x};
                const double x1[7] = {below[k].y, b[1 - line], b[1 - near], own[k].y, b[1 + near], b[1 + line],
                                      above[k].y};
                const uint32_t h0 = have[k] & 0xFFu, h1 = have[k] >> 8;
                double s0, s1;
                if (__all((have[k] | 0x1414u) == 0x7F7Fu)) {
                    s0 = march_row<true>(C, x0, h0);
                    s1 = march_row<true>(C, x1, h1);
                } else {
                    s0 = march_row<false>(C, x0, h0);
                    s1 = march_row<false>(C, x1, h1);
                }
                if (in1) {
                    const dbl2m v{s0, s1};
                    __builtin_memcpy(q + i, &v, 16);
                } else if (in0) {
                    q[i] = s0;
                }
                if (MODE == kSpmvDot) {
                    if (in0) acc = fma(own[k].x, s0, acc);
                    if (in1) acc = fma(own[k].y, s1, acc);
                }
                below[k] = own[k];
                own[k] = above[k];
                above[k] = next[k];
                have[k] = have_next[k];
            }
#pragma unroll
            for (int k = 0; k < kMHalo; ++k) halo[k] = halo_next[k];
        }
        __syncthreads();   // the next item writes the window
    }
    if (MODE == kSpmvPlain) return;
    const double s = block_sum<kMT>(acc, sh);
    if (threadIdx.x == 0) out[blockIdx.x] = s;
}

}  // namespace

// From 6M rows on: us per iteration of plain CG with the gathering kernel and
// with this one, 2.1M rows 37 and 42, 4.1M 59 and 64, 8M 123 and 110, 256^3 286
// and 238, 400 x 400 x 128 347 and 312 (below, the caches hold p and a plane
// has too few tiles to fill the GPU).
bool march_applies(int32_t m, const StenGlobal &C, const double *p, const double *p_own) {
    if (!C.konst || C.width != 7 || m < kMarchRows || (p_own && p_own != p)) return false;
    if (C.offs[3] != 0 || C.offs[4] < 1) return false;
    for (int e = 0; e < 3; ++e)
        if (C.offs[e] != -C.offs[6 - e]) return false;
    // (even: a pair of rows never ends a plane or the vector half way)
    return C.offs[5] <= kMarchLine && C.offs[6] >= 4 * kMTile && C.offs[6] % 2 == 0 && m % 2 == 0;
}

hipError_t launch_spmv_march(int32_t m, const StenGlobal &C, const uint8_t *mask, int grid, const double *p, double *q,
                             double *out, const DevState *st, int mode, hipStream_t s) {
    MarchShape G;
    G.planes = (int32_t)(((int64_t)m + C.offs[6] - 1) / C.offs[6]);
    G.tiles = (C.offs[6] + kMTile - 1) / kMTile;
    // about two workgroups per compute unit, none with less than 8 planes
    const int walks = std::max(1, std::min((512 + G.tiles - 1) / G.tiles, (G.planes + 7) / 8));
    G.walk = (G.planes + walks - 1) / walks;
    G.chunks = (G.planes + G.walk - 1) / G.walk;
    const size_t lds = 2 * sizeof(double) * ((size_t)kMTile + 2 * (size_t)C.offs[5]);
    if (mode == kSpmvPlain)
        hipLaunchKernelGGL((k_spmv_march<kSpmvPlain>), dim3(grid), dim3(kMT), lds, s, m, C, G, mask, p, q, out, st);
    else if (mode == kSpmvDot)
        hipLaunchKernelGGL((k_spmv_march<kSpmvDot>), dim3(grid), dim3(kMT), lds, s, m, C, G, mask, p, q, out, st);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace cgmi
