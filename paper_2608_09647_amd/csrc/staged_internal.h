// Staged column segments (kernels_staged.hip): the layout shared by the
// kernels and the host code that builds it (staged.cpp).
#pragma once
#include <hip/hip_runtime_api.h>
#include <stdint.h>

#include "cgmi_internal.h"

namespace cgmi {

constexpr int kStagedWaves = 16;                     // waves per workgroup
constexpr size_t kStagedLds = 158 * 1024;            // of 160 KB per compute unit
constexpr int kStagedChunks = 4;                     // 16-byte pieces of a segment per thread, at most
constexpr int kStagedAhead = 6;                      // steps of a list loaded ahead, at most
constexpr int kStagedSlack = kStagedAhead * kWaveSize;   // entries past the last list that may be loaded
constexpr int kStagedPerSlot = 4;                    // entries of a row and segment per slot, at most on average
constexpr int kStagedRows = 8192;                    // rows per block aimed at (64 KB of sums)

// An entry's word: column in the segment (15 bits), turn (3), slot of its
// row's sum in the block (14; the slot after the block's last is a dummy).
constexpr int kStagedColBits = 15, kStagedTurnBits = 3;
constexpr uint32_t kStagedTurns = 1u << kStagedTurnBits;
constexpr int kStagedMaxSlots = (1 << (32 - kStagedColBits - kStagedTurnBits)) - 1;
CGMI_HD constexpr inline uint32_t staged_word(uint32_t col, uint32_t turn, uint32_t slot) {
    return col | turn << kStagedColBits | slot << (kStagedColBits + kStagedTurnBits);
}
CGMI_HD constexpr inline uint32_t staged_col(uint32_t w) { return w & ((1u << kStagedColBits) - 1); }
CGMI_HD constexpr inline uint32_t staged_turn(uint32_t w) { return w >> kStagedColBits & (kStagedTurns - 1); }
CGMI_HD constexpr inline uint32_t staged_slot(uint32_t w) { return w >> (kStagedColBits + kStagedTurnBits); }

// LDS of a workgroup: two segments, and the block's slots with the dummy.
CGMI_HD constexpr inline size_t staged_lds(int seg_cols, int max_slots) {
    return sizeof(double) * (2 * (size_t)seg_cols + (size_t)max_slots + 1);
}

// A segment is loaded by 16-byte pairs of columns, pair k of the segment at
// its column k, clamped to the last pair of columns the vector has there (or
// the two behind a whole segment).  `left`: the columns from the segment's
// first to the vector's end, two or more (staged_width; moving the base for a
// segment of one column instead cost the product 1%, 171.2 to 172.5 us for 900K
// rows of 49 entries).
CGMI_HD constexpr inline int32_t staged_last_pair(int32_t left, int32_t seg_cols) {
    return (left < seg_cols + 2 ? left : seg_cols + 2) / 2 * 2 - 2;
}
constexpr int32_t kStagedUnit = 256;                 // a segment's columns are a multiple
// The columns of a segment, at most `widest`: equal parts of as few segments as
// that allows, or fewer columns where the last segment would hold a single one.
// 0: no width does.
inline int32_t staged_width(int32_t ncols, int32_t widest) {
    widest = widest / kStagedUnit * kStagedUnit;
    if (widest <= 0) return 0;
    const int32_t nseg = (int32_t)(((int64_t)ncols + widest - 1) / widest);
    int32_t w = (int32_t)(((int64_t)ncols + nseg - 1) / nseg);
    w = (w + kStagedUnit - 1) / kStagedUnit * kStagedUnit;
    if (w > widest) w = widest;
    while (w > 0 && ncols % w == 1) w -= kStagedUnit;
    return w;
}

struct StagedDev {
    int32_t m;
    int32_t nblocks, ngroups;     // row blocks, groups of segments (a workgroup takes one of each)
    int32_t nseg, seg_cols;       // segments, columns per segment
    int32_t max_slots;            // slots of the longest block
    int32_t ncols;                // columns the vector is known to have
    int32_t ahead;                // steps of the average list, the last one begun counted
    const int32_t *row0;          // [nblocks * kStagedWaves + 1] first row of every wave
    const int32_t *nslots;        // [nblocks] slots of every block
    const int32_t *off;           // [nblocks * kStagedWaves * nseg + 1] first entry of every wave's list per segment
    const uint32_t *idx;          // staged_word of every entry
    const double *val;
    const uint32_t *slots;        // per row: its first slot in the block | its slots << 16; null: one each, in order
    double *part;                 // [ngroups * m] the groups' sums of every row
};

// Lets the kernels use kStagedLds bytes of LDS on the current device.
hipError_t staged_setup();
// The modes of launch_spmv; grid: workgroups of the second kernel, and the
// partials in out (twice that in the residual mode).
hipError_t launch_spmv_staged(const StagedDev &D, int grid, const double *p, double *q, const double *p_own,
                              const double *b, double *p_dst, double *out, Partials in0, Partials in1,
                              DevState *st, int mode, int k0_check, hipStream_t s);

}  // namespace cgmi
