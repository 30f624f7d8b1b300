// host_checks.cpp -- checks of the library's host code without a GPU: the
// host sources (cgmi.cpp, devmatrix.cpp, staged.cpp, fsai.cpp) are linked with
// the HIP calls below, which keep "device" memory on the host, and with
// kernel launches that record what they are asked for or do nothing (those
// that no check reaches stay unresolved).
//
//     host_checks staged ROWS COLS PER_ROW
//         the staged column segments of a matrix of ROWS rows, PER_ROW random
//         entries each (every fifth row twice as many, one row 1500), all
//         columns below COLS: every index the product's kernel forms lies in
//         its buffer, and the sums are the rows' own.  Says whether the
//         schedule runs its products on them
#include <hip/hip_runtime_api.h>

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <string>
#include <vector>

#include "../../paper_2608_09647_amd/csrc/cgmi_host.h"

using namespace cgmi;

// ---------------------------------------------------------------------------
// HIP on host memory

extern "C" {
hipError_t hipMalloc(void **p, size_t n) { return (*p = std::malloc(n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void *p) {
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemset(void *d, int v, size_t n) {
    std::memset(d, v, n);
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error"; }
}

namespace cgmi {
hipError_t staged_setup() { return hipSuccess; }
}

// ---------------------------------------------------------------------------

namespace {

[[noreturn]] void die(const std::string &what) {
    std::printf("FAILED: %s\n", what.c_str());
    std::exit(1);
}
#define REQUIRE(cond, ...)                                   \
    do {                                                     \
        if (!(cond)) {                                       \
            char text_[256];                                 \
            std::snprintf(text_, sizeof text_, __VA_ARGS__); \
            die(std::string(#cond) + ": " + text_);          \
        }                                                    \
    } while (0)

// per_row entries a row, in every fifth row twice as many, in one 1500 (which
// keeps the schedule from stream tiles), one in each of as many equal ranges of
// the columns, integer values (their sums are exact in any order); the last
// column is used.
struct Matrix {
    std::vector<int32_t> rp, ci;
    std::vector<double> val;
};
Matrix random_rows(int32_t rows, int32_t cols, int32_t per_row) {
    Matrix A;
    std::mt19937 rng(7);
    A.rp.assign(1, 0);
    for (int32_t i = 0; i < rows; ++i) {
        const int32_t len = i == rows / 2 ? 1500 : i % 5 ? per_row : 2 * per_row, width = cols / len;
        REQUIRE(width > 0, "%d columns for %d entries a row", cols, len);
        for (int32_t j = 0; j < len; ++j) {
            A.ci.push_back(j * width + (int32_t)(rng() % (uint32_t)width));
            A.val.push_back((double)(int32_t)(rng() % 17u) - 8.0);
        }
        A.rp.push_back((int32_t)A.ci.size());
    }
    A.ci.back() = cols - 1;
    return A;
}

// The product of the staged layout S, entry by entry with the indices the
// kernel forms: list bounds, entry loads (those ahead too), the pieces of p
// staged for every thread, columns and slots in LDS.
std::vector<double> staged_product(const StagedDev &S, const std::vector<double> &p, size_t entries) {
    constexpr int threads = kStagedWaves * kWaveSize, E = 16 / (int)sizeof(double);
    const int chunks = (S.seg_cols * (int)sizeof(double) / 16 + threads - 1) / threads <= 3 ? 3 : 4;
    REQUIRE(S.nseg >= 2 && S.seg_cols % 256 == 0 && S.seg_cols * (int)sizeof(double) <= 16 * threads * kStagedChunks,
            "%d segments of %d", S.nseg, S.seg_cols);
    REQUIRE(staged_lds(S.seg_cols, S.max_slots) <= kStagedLds, "%d columns, %d slots", S.seg_cols, S.max_slots);
    REQUIRE((int64_t)(S.nseg - 1) * S.seg_cols < S.ncols && (int64_t)S.nseg * S.seg_cols >= S.ncols,
            "%d segments of %d for %d columns", S.nseg, S.seg_cols, S.ncols);
    // what segment_load reads, and what segment_store leaves in LDS
    std::vector<std::vector<double>> lds((size_t)S.nseg, std::vector<double>((size_t)S.seg_cols, NAN));
    for (int32_t seg = 0; seg < S.nseg + 2; ++seg) {
        const int32_t s = std::min(seg, S.nseg - 1);
        const int64_t first = (int64_t)s * S.seg_cols;
        for (int32_t u = 0; u < chunks; ++u)
            for (int32_t t = 0; t < threads; ++t) {
                const int32_t k = (u * threads + t) * E;
                int64_t at = first + k;
                if (!(seg < S.nseg - 1 && S.seg_cols == chunks * threads * E)) {
                    const int32_t last = staged_last_pair(S.ncols - s * S.seg_cols, S.seg_cols);
                    at = first + staged_pair_base(last) + (int64_t)staged_pair(k, last);
                }
                REQUIRE(at >= 0 && at + E <= S.ncols, "segment %d of %d reads p[%lld] of %d", (int)seg, S.nseg,
                        (long long)at, S.ncols);
                if (seg < S.nseg && k < S.seg_cols)
                    for (int e = 0; e < E; ++e) lds[(size_t)seg][(size_t)(k + e)] = p[(size_t)(at + e)];
            }
        if (seg == S.nseg - 1)
            for (int32_t c = S.ncols / E * E; c < S.ncols; ++c) {
                REQUIRE(c - first >= 0 && c - first < S.seg_cols, "tail column %d of segment %d", c, seg);
                lds[(size_t)seg][(size_t)(c - first)] = p[(size_t)c];
            }
    }
    const size_t lists = (size_t)S.nblocks * kStagedWaves * S.nseg;
    REQUIRE(S.off[0] == 0 && (size_t)S.off[lists] <= entries, "%d entries", S.off[lists]);
    std::vector<double> q((size_t)S.m, 0.0);
    for (int32_t b = 0; b < S.nblocks; ++b)
        for (int32_t g = 0; g < S.ngroups; ++g) {
            std::vector<double> y((size_t)S.nslots[b] + 1, 0.0);
            REQUIRE(S.nslots[b] <= S.max_slots, "block %d", b);
            const int32_t first = (int32_t)((int64_t)S.nseg * g / S.ngroups);
            const int32_t last = (int32_t)((int64_t)S.nseg * (g + 1) / S.ngroups);
            REQUIRE(first < last, "group %d of %d has no segment (of %d)", g, S.ngroups, S.nseg);
            for (int w = 0; w < kStagedWaves; ++w)
                for (int32_t s = first; s < last; ++s) {
                    const size_t l = ((size_t)b * kStagedWaves + w) * S.nseg + s;
                    const int32_t beg = S.off[l], end = S.off[l + 1];
                    REQUIRE(beg >= 0 && beg <= end && (size_t)beg + kStagedSlack <= entries, "list %zu", l);
                    for (int32_t k = beg; k < end; ++k) {
                        const uint32_t col = staged_col(S.idx[k]), slot = staged_slot(S.idx[k]);
                        REQUIRE((int)slot <= S.nslots[b], "slot %u of %d", slot, S.nslots[b]);
                        REQUIRE((int)col < S.seg_cols, "column %u", col);
                        if ((int)slot < S.nslots[b]) y[slot] += S.val[k] * lds[(size_t)s][col];
                    }
                }
            for (int32_t r = S.row0[(size_t)b * kStagedWaves]; r < S.row0[((size_t)b + 1) * kStagedWaves]; ++r) {
                const uint32_t u = S.slots ? S.slots[r] : (uint32_t)(r - S.row0[(size_t)b * kStagedWaves]) | 1u << 16;
                for (uint32_t i = 0; i < u >> 16; ++i) q[(size_t)r] += y[(u & 0xFFFFu) + i];
            }
        }
    return q;
}

void check_staged(int32_t rows, int32_t cols, int32_t per_row) {
    const int cus = 256;
    const Matrix A = random_rows(rows, cols, per_row);
    DevMatrix M;
    REQUIRE(dm_upload(M, rows, A.rp.data(), A.ci.data(), A.val.data(), 0) == CG_OK, "upload");
    REQUIRE(dm_schedule(M, 0, 0, cus, 16 * cus, false) == CG_OK, "schedule");
    std::printf("%s ", M.use_st64 ? "taken" : "not taken");
    if (M.st64.state == 0) staged_build(M, cus, M.st64);
    if (M.st64.state < 0) {
        std::printf("not built\n");
        dm_free(M);
        return;
    }
    const StagedDev &S = M.st64.dev;
    std::printf("groups %d segments %d of %d columns, %d in the last\n", S.ngroups, S.nseg, S.seg_cols,
                S.ncols - (S.nseg - 1) * S.seg_cols);
    REQUIRE(S.ncols == cols && S.m == rows, "%d x %d", S.m, S.ncols);
    std::vector<double> p((size_t)cols);
    std::mt19937 rng(9);
    for (double &v : p) v = (double)(int32_t)(rng() % 17u) - 8.0;
    const std::vector<double> q = staged_product(S, p, (size_t)(M.nnz + M.nnz / 8) + kStagedSlack);
    for (int32_t i = 0; i < rows; ++i) {
        double s = 0.0;
        for (int32_t k = A.rp[(size_t)i]; k < A.rp[(size_t)i + 1]; ++k)
            s += A.val[(size_t)k] * p[(size_t)A.ci[(size_t)k]];
        REQUIRE(s == q[(size_t)i], "row %d: %g, not %g", i, q[(size_t)i], s);
    }
    dm_free(M);
}

}  // namespace

int main(int argc, char **argv) {
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "staged" && argc == 5) check_staged(std::atoi(argv[2]), std::atoi(argv[3]), std::atoi(argv[4]));
    else die("usage: host_checks staged ROWS COLS PER_ROW");
    std::printf("ok\n");
    return 0;
}
